// A filter in MFMA fragment order, one block of 256 threads per 32-row block and 16-channel block: a piece of work that
// shares a launch with others (the input repack and the slice sum in conv_mfma.hip, the pooling in compress.hip).
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

__device__ __forceinline__ void filter_repack(const FilterRepack &p, const int b, bf16_t *sm)
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
    const int L = cols * p.RS, Lp = L + 2;
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    // a wave takes every fourth row; all of a thread's loads are issued before the first is
    // used (at most 8 rows of 3 x 64 elements, or 4 rows of 5 x 64)
    constexpr int kRowsPerWave = 8, kMaxX = 5;
    const rsrc_t rs = make_rsrc(p.W, (uint32_t)p.O * p.Cw * p.RS * 2u);
    // Whole blocks whose runs are multiples of 16 bytes and start on such (every row of W does
    // when Cw * RS is a multiple of 8): 16-byte loads, at most 3 per thread, instead of up to 40
    // loads of one element each.
    const int segs = L >> 3;
    if ((L & 7) == 0 && ((p.Cw * p.RS) & 7) == 0 && c0 + cols <= p.Cw) {
        u32x4 t4[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int it = threadIdx.x + 256 * q, r = it / segs, sg = it - r * segs, o = o0 + r;
            const bool ok = it < rows * segs && o < p.O;
            t4[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, ok ? ((uint32_t)(o * p.Cw + c0) * p.RS) * 2u + sg * 16u : kNoLoad, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int it = threadIdx.x + 256 * q, r = it / segs, sg = it - r * segs;
            if (it < rows * segs) {
                uint32_t *d = (uint32_t *)(sm + r * Lp + sg * 8); // (Lp is even: 4-byte aligned)
#pragma unroll
                for (int k = 0; k < 4; ++k) d[k] = t4[q][k];
            }
        }
    } else {
    uint16_t tmp[kRowsPerWave][kMaxX];
#pragma unroll
    for (int j = 0; j < kRowsPerWave; ++j) {
        const int r = wv + 4 * j, o = o0 + r;
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
        const int r = wv + 4 * j;
#pragma unroll
        for (int k = 0; k < kMaxX; ++k) {
            const int x = ln + 64 * k;
            if (r < rows && x < L) sm[r * Lp + x] = tmp[j][k];
        }
    }
    }
    __syncthreads();
    for (int it = threadIdx.x; it < p.RS * 64; it += 256) {
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

} // namespace cac
