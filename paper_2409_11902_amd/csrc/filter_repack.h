// What a convolution's operands need ahead of it, in blocks of 256 threads: a filter in MFMA fragment order, one block per
// 32-row block and 16-channel block, and the channels-last copy of an input.  Pieces of work that share a launch with others
// (the pooling in compress.hip, the weight gradient in dw_mfma.hip) or have one (repack_kernel in conv_mfma.hip).
#pragma once
#include "common.h"

namespace cac {

// W [O][Cw][RS taps] -> Wt [RS][KCp/16][Mp/32][lane 64][8]: lane l of a wave holds row m = 32*mblk + l%32 and the 8
// channels kc = 16*kblk + 8*(l/32) ..., so a wave reads the A fragment of a (tap, 16-channel block, 32-row block) as one
// contiguous KiB.  Forward: m = o, kc = c; transpose (data gradient): m = c, kc = o.
struct FilterRepack {
    const bf16_t *W;
    bf16_t *Wt;
    int O, Cw, RS, Mp, KCp, transpose;
    unsigned blocks() const { return (unsigned)((Mp / 32) * (KCp / 16)); }
};
constexpr int kFilterElems = 32 * (16 * 9 + 2); // LDS: a 32 x 16 block of (o, c) pairs, 9 taps, padded rows

// NT threads, 256 or one wave, by themselves.
template <int NT> __device__ __forceinline__ void filter_repack_by(const FilterRepack &p, const int b, bf16_t *sm, const int tid)
{
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    constexpr uint32_t kNoLoad = 0x80000000u;
    // One block per (32-row block, 16-channel block): its part of W -- for every o a contiguous
    // run of (c, tap) -- goes through LDS as it lies in memory; then every thread gathers the
    // 8 channels of one lane of one tap's fragment and writes them as 16 bytes, a wave one
    // contiguous KiB.  Rows are padded to an odd number of dwords against bank conflicts.
    const int mblks = p.Mp / 32, kblks = p.KCp / 16, mblk = b % mblks, kblk = b / mblks;
    const int rows = p.transpose ? 16 : 32, cols = p.transpose ? 32 : 16; // o rows, c columns
    const int o0 = p.transpose ? kblk * 16 : mblk * 32, c0 = p.transpose ? mblk * 32 : kblk * 16;
    // (A wave has rows past the last channel left out: they are of outputs that nobody stores, and as the partial block that they are,
    // read element by element, they held it up by 4-7 us.)
    if (NT == 64 && p.transpose && c0 >= p.Cw) return;
    const int L = cols * p.RS, Lp = L + 2;
    const int wv = tid >> 6, ln = tid & 63;
    // a wave takes every fourth row; all of a thread's loads are issued before the first is
    // used (at most 8 rows of 3 x 64 elements, or 4 rows of 5 x 64; a wave by itself: 8 rows at a time)
    constexpr int kRowsPerWave = 8, kMaxX = 5, kWaves = NT / 64;
    const rsrc_t rs = make_rsrc(p.W, (uint32_t)p.O * p.Cw * p.RS * 2u);
    // Whole blocks whose runs are multiples of 16 bytes and start on such (every row of W does
    // when Cw * RS is a multiple of 8): 16-byte loads, at most 3 per thread, instead of up to 40
    // loads of one element each.
    const int segs = L >> 3;
    if ((L & 7) == 0 && ((p.Cw * p.RS) & 7) == 0 && c0 + cols <= p.Cw) {
        constexpr int kLoads = 768 / NT;
        u32x4 t4[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const int it = tid + NT * q, r = it / segs, sg = it - r * segs, o = o0 + r;
            const bool ok = it < rows * segs && o < p.O;
            t4[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, ok ? ((uint32_t)(o * p.Cw + c0) * p.RS) * 2u + sg * 16u : kNoLoad, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const int it = tid + NT * q, r = it / segs, sg = it - r * segs;
            if (it < rows * segs) {
                uint32_t *d = (uint32_t *)(sm + r * Lp + sg * 8); // (Lp is even: 4-byte aligned)
#pragma unroll
                for (int k = 0; k < 4; ++k) d[k] = t4[q][k];
            }
        }
    } else {
    for (int r0 = 0; r0 < 32; r0 += kRowsPerWave * kWaves) {
    uint16_t tmp[kRowsPerWave][kMaxX];
#pragma unroll
    for (int j = 0; j < kRowsPerWave; ++j) {
        const int r = r0 + wv + kWaves * j, o = o0 + r;
        const int lim = (r < rows && o < p.O) ? min(L, (p.Cw - c0) * p.RS) : 0; // elements of the run inside the tensor
        const uint32_t base = ((uint32_t)(o * p.Cw + c0) * p.RS) * 2u;
#pragma unroll
        for (int k = 0; k < kMaxX; ++k) {
            const int x = ln + 64 * k;
            tmp[j][k] = __builtin_amdgcn_raw_buffer_load_b16(rs, x < lim ? base + 2u * x : kNoLoad, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < kRowsPerWave; ++j) {
        const int r = r0 + wv + kWaves * j;
#pragma unroll
        for (int k = 0; k < kMaxX; ++k) {
            const int x = ln + 64 * k;
            if (r < rows && x < L) sm[r * Lp + x] = tmp[j][k];
        }
    }
    }
    }
    if constexpr (NT > 64) {
        __syncthreads();
    } else { // (a wave reads what it wrote itself: LDS serves a wave's requests in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    for (int it = tid; it < p.RS * 64; it += NT) {
        const int tap = it >> 6, lane = it & 63, m = lane & 31, k8 = 8 * (lane >> 5);
        u32x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t h[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int kc = k8 + 2 * k + e;
                h[e] = p.transpose ? sm[kc * Lp + m * p.RS + tap] : sm[m * Lp + kc * p.RS + tap];
            }
            v[k] = h[0] | (h[1] << 16);
        }
        ((u32x4 *)p.Wt)[((long)(tap * kblks + kblk) * mblks + mblk) * 64 + lane] = v;
    }
}

__device__ __forceinline__ void filter_repack(const FilterRepack &p, const int b, bf16_t *sm, const int tid) { filter_repack_by<256>(p, b, sm, tid); }
__device__ __forceinline__ void filter_repack_wave(const FilterRepack &p, const int b, bf16_t *sm, const int lane)
{
    filter_repack_by<64>(p, b, sm, lane);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); // (the next block goes to the same place)
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Both repacks of a call, and zeros.
//
// Input: in [N][C][HW] -> out [N][HW][Cp], zeros for c >= C.
//   HW even (every plane starts at a multiple of 4 bytes): a thread moves an 8 channel x 8 pixel
//   block: eight 16-byte loads along the pixels (consecutive lanes = consecutive pixel groups of
//   a channel row), an 8 x 8 transpose in registers (v_perm), eight 16-byte stores of 8 channels
//   each; the last block of a plane may be partial (it reads on into the next plane, or zeros
//   past the tensor, and stores only its own pixels).
//   Otherwise: 64 x 64 tiles through LDS, element by element.
// Blocks [0, in_blocks) do the input, then filter.blocks() the filter, the rest the zeros.
struct RepackParams {
    const bf16_t *in;
    bf16_t *out;        // null: no channels-last copy, the input blocks only form Z
    int N, C, HW, Cp, in_blocks, fast;
    int in_wpb;         // waves of an input block that take items (fast path): fewer than 4 spread a small
                        // input over more compute units, one block each
    bf16_t *Z;          // pooled copy of `in` written on the way (2 x 2 means), or null
    int Wimg;           // image width (only with Z)
    int decim;          // with Z: `out` takes pixel (2h, 2w) of every 2 x 2 tile only, as an image of half the extent
    FilterRepack f;
    bf16_t *zero;       // zero_n elements to clear, 2048 to a block (zero_n 0: none)
    long zero_n;
    unsigned blocks() const { return in_blocks + f.blocks() + (zero_n ? (unsigned)((zero_n / 8 + 256) / 256) : 0u); }
};

constexpr int kRepackElems = kFilterElems > 64 * 66 ? kFilterElems : 64 * 66; // LDS of a block
__device__ __forceinline__ void repack_body(const RepackParams &p, const int bid, bf16_t *sm, const int tid)
{
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    constexpr uint32_t kNoLoad = 0x80000000u;
    if (bid >= p.in_blocks) {
        const int fb = (p.f.Mp / 32) * (p.f.KCp / 16);
        if (bid - p.in_blocks < fb) {
            filter_repack(p.f, bid - p.in_blocks, sm, tid);
        } else if (p.zero_n) { // whole 16-byte units, then the (up to 7) elements that remain -- not a byte past the tensor
            const long i = (long)(bid - p.in_blocks - fb) * 256 + tid, n16 = p.zero_n / 8;
            if (i < n16) ((u32x4 *)p.zero)[i] = u32x4{0, 0, 0, 0};
            if (i < p.zero_n - n16 * 8) p.zero[n16 * 8 + i] = (bf16_t)0;
        }
        return;
    }
    bf16_t (*tile)[66] = (bf16_t (*)[66])sm;
    if (p.fast) {
        // item -> (image n, block of up to 8 channel groups, pixel group pg of 8, channel group
        // within the block), the last fastest: 8 neighbouring lanes read 8 channel rows and
        // write the 128 contiguous bytes of 64 channels of one pixel; the next lanes move along
        // the pixels, so every row is read in 128-byte runs too.  With Z, an item is the same 8
        // pixels of TWO image rows (2h, 2h+1), from which it also forms the 2 x 2 means.
        const bool pool = p.Z != nullptr && p.Wimg != 4;
        const bool pool4 = p.Z != nullptr && p.Wimg == 4; // rows of 4 pixels: an item is already two whole rows
        const int wgs = pool ? p.Wimg / 8 : 1;                 // pixel groups per image row
        const int pgs = pool ? p.HW / 16 : (p.HW + 7) / 8;     // items along the pixels (the last may be partial)
        const int cgs = p.Cp / 8, cgw = min(cgs, 8), cgb = (cgs + cgw - 1) / cgw;
        if ((int)(tid >> 6) >= p.in_wpb) return;
        // (fewer than 2^31 items: 32-bit divisions)
        const uint32_t item = ((uint32_t)bid * p.in_wpb + (tid >> 6)) * 64u + (tid & 63);
        if (item >= (uint32_t)p.N * cgb * pgs * cgw) return;
        const int cl = item % (uint32_t)cgw;
        uint32_t t1 = item / (uint32_t)cgw;
        const int pi = t1 % (uint32_t)pgs;
        t1 /= (uint32_t)pgs;
        const int cg = (int)(t1 % (uint32_t)cgb) * cgw + cl, n = t1 / (uint32_t)cgb;
        if (cg >= cgs) return;
        // first pixel of the item's (first) row segment
        const int hh = pool ? pi / wgs : 0, wg = pool ? pi - hh * wgs : 0;
        const int px0 = pool ? (2 * hh * wgs + wg) * 8 : pi * 8;
        const rsrc_t rs = make_rsrc(p.in, (uint32_t)p.N * p.C * p.HW * 2u);
        u32x4 r[2][8];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if (a == 1 && !pool) break;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = cg * 8 + i;
                const uint32_t e = ((uint32_t)(n * p.C + c) * p.HW + px0 + a * p.Wimg) * 2u;
                r[a][i] = __builtin_amdgcn_raw_buffer_load_b128(rs, c < p.C ? e : kNoLoad, 0, 0);
            }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if (a == 1 && !pool) break;
            if (!p.out) break; // only the pooled map is wanted
            if (p.decim && a == 1) break; // (odd rows are not kept)
            bf16_t *dst = p.decim ? p.out + ((long)n * (p.HW / 4) + hh * (p.Wimg / 2) + wg * 4) * p.Cp + cg * 8
                                  : p.out + ((long)n * p.HW + px0 + a * p.Wimg) * p.Cp + cg * 8;
#pragma unroll
            for (int px = 0; px < 8; ++px) {
                // pixel px of the 8 channels: half px%2 of dword px/2 of every row
                u32x4 v;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t lo = r[a][2 * k][px / 2], hi = r[a][2 * k + 1][px / 2];
                    v[k] = (px & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                }
                if (p.decim) {
                    if (!(px & 1)) *(u32x4 *)(dst + (long)(px / 2) * p.Cp) = v;
                } else if (px0 + px < p.HW) {
                    *(u32x4 *)(dst + (long)px * p.Cp) = v; // (a plane's last item may reach past it)
                }
            }
        }
        if (pool4) {
            // Z[n][c][pi][0..1] from pixels (0, 1, 4, 5) and (2, 3, 6, 7) of the item, summed row by
            // row like the stand-alone kernel does
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = cg * 8 + i;
                if (c >= p.C) break;
                uint32_t h2[2];
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                    const uint32_t t0 = r[0][i][jj], t1r = r[0][i][2 + jj];
                    float sum = 0.f;
                    sum += __uint_as_float(t0 << 16);
                    sum += __uint_as_float(t0 & 0xffff0000u);
                    sum += __uint_as_float(t1r << 16);
                    sum += __uint_as_float(t1r & 0xffff0000u);
                    h2[jj] = f32_to_bf16(sum * 0.25f);
                }
                *(uint32_t *)(p.Z + (((long)n * p.C + c) * (p.HW / 8) + pi) * 2) = h2[0] | (h2[1] << 16);
            }
        }
        if (pool) {
            // Z[n][c][hh][4*wg .. +3]: the same sum order and rounding as the stand-alone kernel
            const int Hp = p.HW / p.Wimg / 2, Wp = p.Wimg / 2;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = cg * 8 + i;
                if (c >= p.C) break;
                uint32_t o[2];
#pragma unroll
                for (int j2 = 0; j2 < 2; ++j2) {
                    uint32_t h2[2];
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) {
                        const uint32_t t0 = r[0][i][2 * j2 + jj], t1r = r[1][i][2 * j2 + jj];
                        float sum = 0.f;
                        sum += __uint_as_float(t0 << 16);
                        sum += __uint_as_float(t0 & 0xffff0000u);
                        sum += __uint_as_float(t1r << 16);
                        sum += __uint_as_float(t1r & 0xffff0000u);
                        h2[jj] = f32_to_bf16(sum * 0.25f);
                    }
                    o[j2] = h2[0] | (h2[1] << 16);
                }
                typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
                *(u32x2 *)(p.Z + (((long)n * p.C + c) * Hp + hh) * Wp + wg * 4) = u32x2{o[0], o[1]};
            }
        }
        return;
    }
    // block -> (image, 64-channel block, 64-pixel block)
    const int pbs = (p.HW + 63) / 64, cbs = (p.Cp + 63) / 64;
    const int pb = bid % pbs, t1 = bid / pbs;
    const int cb = t1 % cbs, n = t1 / cbs;
    const int c0 = cb * 64, p0 = pb * 64;
    const int tx = tid & 63, ty = tid >> 6;
    for (int k = ty; k < 64; k += 4) {
        const int c = c0 + k, px = p0 + tx;
        tile[k][tx] = (c < p.C && px < p.HW && n < p.N) ? p.in[((long)n * p.C + c) * p.HW + px] : (bf16_t)0;
    }
    __syncthreads();
    for (int k = ty; k < 64; k += 4) {
        const int px = p0 + k, c = c0 + tx;
        if (px < p.HW && c < p.Cp && n < p.N) p.out[((long)n * p.HW + px) * p.Cp + c] = tile[tx][k];
    }
}

} // namespace cac
