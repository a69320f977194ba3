// 1 x 1 stride-1 convolution, forward and data gradient, as a GEMM on the tensors as they lie:
//   out[n][m][px] = bias[m] + sum_k W'[m][k] * in[n][k][px],   px over the whole plane (rows do not matter).
//
// These layers are bound by HBM (256 -> 64 at 56 x 56, batch 64: 129 MB for 6.6 GFLOP).  The gather launches of
// conv_mfma.hip write and read a channels-last copy of the input first (forward with a 2 x 2 pooled record: 37 us
// for the copy alone on that layer) and have two MFMA steps per 32 channels to hide anything behind.  Here a
// workgroup of four waves owns 64 or 128 output channels x 256 pixels and goes through the input in stages of 64
// channels:
//   - a thread moves one item of 8 channels x 8 pixels per stage -- eight loads, the next stage's always in flight
//     while this one is multiplied --, transposes it in registers and writes it to one of two LDS buffers as
//     [pixel][channel]; the lanes of a wave lie along the pixels (along the channels, every lane is a cache access of
//     its own: 57 instead of 41 us on the layer above, the vector cache busy throughout);
//   - the filter fragments of a stage are all requested before the next stage's input, so that waiting for them
//     does not mean waiting for HBM (loads return in order);
//   - with a 2 x 2 mean record over rows of a multiple of 4 pixels an item is 8 channels x 2 rows x 4 pixels, and
//     the thread pools what it holds: Z costs its own bytes only (same sum order and rounding as the stand-alone
//     kernel, bit-identical);
//   - the result leaves through LDS as in conv_tile.hip.
// Per call (bench layers, batch 64, inputs resident): 256 -> 64 at 56 x 56 forward 74 -> 39 us, 64 -> 256 61 -> 39, their data
// gradients 53 -> 34 and 49 -> 29 (small maps: conv_pw_wave_kernel below).  Two stages of input in flight (for 64
// channels per workgroup, which have the registers) measured 2-10 % slower: the stages are not bound by latency.
#include <stdio.h>
#include <stdlib.h>

#include <mutex>
#include <type_traits>

#include "common.h"
#include "conv_mfma.h"
#include "tile_stage.h"

namespace cac {

namespace {

using namespace tile;

constexpr int KC = 64, KCS = KC + 8, KSTEPS = KC / 16;
constexpr int kPT = 256, kGroups = kPT / 8; // pixels of a tile; items along the pixels
constexpr int kEpRow = 64 * 2 + 16, kEpWave = 32 * kEpRow;
constexpr int kBuf = kPT * KCS * 2 + kPT / 4 * 16; // (with the largest padding, see pad_of)

// FUSE: items of 2 rows x 4 pixels, Z written on the way.  GW: pixels of an item otherwise: 8, or 7 for planes of odd
// size (read from the dword below an odd start).  EPI: pixels per store.  TAIL: the launch may have workgroups that add a weight
// gradient's slices (here and below a form of its own: forward passes of 1056 -> 976 at 4 x 4, batch 1, 9.2 us with the branch, 8.7 without).
template <int NI, int WM, int WN, bool FUSE, int GW, int EPI, bool TAIL>
__global__ void __launch_bounds__(256, 2) conv_pw_kernel(GatherParams p)
{
    constexpr int MI = 2;
    static_assert(WN * NI * 32 == kPT && WM * WN == 4, "");
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    unsigned bx = blockIdx.x, by = blockIdx.y, bz = 0;
    if constexpr (TAIL) {
        if (!conv_block(p, smem, bx, by, bz)) return;
    }
    const int tau = bx % p.tiles_per_img, n_base = bx / p.tiles_per_img * p.IPT;
    const int ppi = p.Hc * p.Wc, K = p.KCin, nkb = p.nkb;
    const int pix0 = p.IPT > 1 ? 0 : tau * p.tile_px;
    const int m0 = (by * WM + wm) * 64;

    // ---- this thread's item: 8 channels, pixels from px0 on of image n_base + ig
    // (lanes along the pixels: a wave's load then covers whole lines of one or two channel rows; with the lanes along the
    // channels every lane was a cache access of its own, 64 to the load, and the vector cache bound the kernel)
    const int gidx = tid % kGroups, oct = tid / kGroups;
    // LDS: 16 bytes more after every 8 (4) pixels, so that the items of neighbouring lanes start in different banks
    auto pad_of = [](int px) { return FUSE ? (px >> 2) * 16 : GW == 8 ? (px >> 3) * 16 : 0; };
    int ig = 0, px0, lpx; // first pixel in the plane; in LDS
    bool item = true;
    if constexpr (FUSE) {
        const int pair = fdiv(gidx, p.m_gx), c4 = gidx - pair * p.GX;
        lpx = pair * 2 * p.Win + c4 * 4;
        px0 = pix0 + lpx;
        item = lpx < p.tile_px && px0 < ppi;
    } else {
        ig = p.IPT > 1 ? fdiv(gidx, p.m_gx) : 0;
        const int gx = gidx - ig * p.GX;
        px0 = pix0 + gx * GW;
        lpx = gidx * GW;
        item = ig < p.IPT && px0 < ppi;
    }
    item = item && n_base + ig < p.N;
    const uint32_t e0 = item ? (uint32_t)((n_base + ig) * K + oct * 8) * ppi + px0 : kNoElem;
    const uint32_t l0 = lds0 + (uint32_t)(lpx * KCS + oct * 8) * 2u + pad_of(lpx);
    const rsrc_t rs_in = make_rsrc(p.in, (uint32_t)p.N * K * ppi * 2u);
    typedef std::conditional_t<FUSE, u32x2, u32x4> item_t;
    constexpr int ROWS = FUSE ? 2 : 1;
    item_t r[8][ROWS];
    auto fetch = [&](int s) {
        uint32_t e = e0 + (uint32_t)(s * KC) * ppi;
        opaque(e);
        const int nvalid = K - (s * KC + oct * 8); // channels that exist (none past the last stage)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t ei = i < nvalid ? e : kNoElem;
            if constexpr (FUSE) {
                r[i][0] = __builtin_amdgcn_raw_buffer_load_b64(rs_in, ei * 2u, 0, 0);
                r[i][1] = __builtin_amdgcn_raw_buffer_load_b64(rs_in, (ei + p.Win) * 2u, 0, 0);
            } else {
                r[i][0] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, (GW == 7 ? ei & ~1u : ei) * 2u, 0, 0);
            }
            e += ppi;
        }
    };
    // the item of stage s: Z, then to LDS
    const rsrc_t rs_z = make_rsrc(p.Z, (uint32_t)p.N * K * (ppi / 4) * 2u);
    auto put = [&](int s, uint32_t buf) {
        if (!item) return; // (the pixels of items that do not exist are never stored, whatever LDS holds for them)
        if constexpr (FUSE) {
            if (by == 0) {
                const int nvalid = K - (s * KC + oct * 8);
                // plane * (ppi / 4) + pooled row * Wp + pooled column; px0 = 2 * pooled row * W + 2 * pooled column
                const int prow = fdiv(px0, p.m_w2), pcol = (px0 - prow * 2 * p.Win) >> 1;
                uint32_t z = ((uint32_t)(n_base * K + s * KC + oct * 8) * (ppi / 4) + prow * (p.Win / 2) + pcol) * 2u;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    uint32_t h[2];
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) {
                        const uint32_t t0 = r[i][0][jj], t1 = r[i][1][jj];
                        float sum = 0.f;
                        sum += __uint_as_float(t0 << 16);
                        sum += __uint_as_float(t0 & 0xffff0000u);
                        sum += __uint_as_float(t1 << 16);
                        sum += __uint_as_float(t1 & 0xffff0000u);
                        h[jj] = f32_to_bf16(sum * 0.25f);
                    }
                    __builtin_amdgcn_raw_buffer_store_b32(h[0] | (h[1] << 16), rs_z, i < nvalid ? z : kNoLoad, 0, 0);
                    z += (uint32_t)(ppi / 4) * 2u;
                }
            }
        }
        if constexpr (GW == 7) {
            const uint32_t par = e0 + (uint32_t)(s * KC) * ppi;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t sh = ((par + i * ppi) & 1u) * 16u;
                auto &v = r[i][0];
#pragma unroll
                for (int k = 0; k + 1 < (int)(sizeof(item_t) / 4); ++k) v[k] = __builtin_amdgcn_alignbit(v[k + 1], v[k], sh);
                v[sizeof(item_t) / 4 - 1] >>= sh;
            }
        }
#pragma unroll
        for (int a = 0; a < ROWS; ++a)
#pragma unroll
            for (int px = 0; px < (FUSE ? 4 : GW); ++px) {
                u32x4 v; // pixel px of the 8 channels
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t lo = r[2 * k][a][px / 2], hi = r[2 * k + 1][a][px / 2];
                    v[k] = (px & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                }
                *(lds_u32x4_ptr)(uintptr_t)(l0 + buf + (a ? p.Win * (KCS * 2) + pad_of(p.Win) : 0) + px * (KCS * 2)) = v;
            }
    };

    // ---- this lane's pixels
    uint32_t pbase[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int idx = (wn * NI + ni) * 32 + l32;
        pbase[ni] = lds0 + 16u * half + (uint32_t)(idx * KCS * 2 + pad_of(idx));
    }
    // ---- filter fragments: offset of the lane, of a 16-channel step, of a block of 32 output channels
    const rsrc_t rs_w = make_rsrc(p.wt, p.w_bytes);
    const uint32_t wlane = p.w_direct ? (m0 + l32 < p.M ? (uint32_t)((m0 + l32) * K + 8 * half) * 2u : kNoLoad)
                                      : (m0 < p.Mp ? (uint32_t)(m0 >> 5) * kFrag + lane * 16u : kNoLoad);
    const uint32_t wlane1 = p.w_direct ? (m0 + 32 + l32 < p.M ? (uint32_t)((m0 + 32 + l32) * K + 8 * half) * 2u : kNoLoad)
                                       : (m0 < p.Mp ? (uint32_t)((m0 >> 5) + 1) * kFrag + lane * 16u : kNoLoad);
    const int ksteps_all = p.KCp / 16;

    f32x16 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[mi][ni][j] = 0.f;
    u32x4 w[KSTEPS][MI];
    auto fetch_w = [&](int s, int kk) {
        // (16-channel steps past the last one: zeros)
        const int step = s * KSTEPS + kk;
        const uint32_t so = (uint32_t)min(step, ksteps_all - 1) * p.w_kstep;
        w[kk][0] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, step < ksteps_all ? wlane : kNoLoad, so, 0);
        w[kk][1] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, step < ksteps_all ? wlane1 : kNoLoad, so, 0);
    };
    fetch(0);
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) fetch_w(0, kk);
    put(0, 0);
    fetch(1);
    __syncthreads();
    for (int s = 0; s < nkb; ++s) {
        const uint32_t buf = (s & 1) ? kBuf : 0u, nbuf = kBuf - buf;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                union { u32x4 u; bf16x8 v; } a0, a1, b;
                b.u = lds16(pbase[ni] + buf + 32 * kk);
                a0.u = w[kk][0];
                a1.u = w[kk][1];
                acc[0][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b.v, a0.v, acc[0][ni], 0, 0, 0);
                acc[1][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b.v, a1.v, acc[1][ni], 0, 0, 0);
            }
            fetch_w(s + 1, kk); // (behind the input of stage s + 1, ahead of that of stage s + 2)
        }
        if (s + 1 < nkb) {
            put(s + 1, nbuf);
            fetch(s + 2); // (past the end: nothing is loaded)
        }
        __syncthreads();
    }
    // ---- epilogue: bias, bfloat16; two pixel blocks x 32 channels at a time through LDS as [channel][pixel] rows, every
    // wave in a part of its own
    const uint32_t plane_out = (uint32_t)ppi;
    const rsrc_t rs_out = make_rsrc(p.out, (uint32_t)p.N * p.M * plane_out * 2u);
    const uint32_t ep = lds0 + wave * kEpWave;
    uint32_t el = lane;
    opaque(el);
    const uint32_t eh = el >> 5, e32 = el & 31;
    float bias[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int m = m0 + mi * 32 + e32;
        bias[mi] = (p.bias && m < p.M) ? bf16_to_f32(p.bias[m]) : 0.f;
    }
    constexpr int LPR = 64 / EPI, RPI = 64 / LPR; // lanes of a row; rows per pass over the lanes
#pragma unroll
    for (int pass = 0; pass < NI / 2; ++pass) {
        const int seg = el % LPR, idx = (wn * NI + pass * 2) * 32 + seg * EPI;
        int g = 0, px = pix0 + idx;
        if (p.IPT > 1) { // (an image's pixels in LDS are whole items)
            g = fdiv(idx, p.m_ppi);
            px = idx - g * (p.GX * GW);
        }
        const int n = n_base + g;
        const bool px_ok = (px < ppi) & (g < p.IPT) & (n < p.N) & (p.IPT > 1 || idx < p.tile_px);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                const f32x16 &a = acc[mi][pass * 2 + nb];
                const float bb = bias[mi];
#pragma unroll
                for (int jq = 0; jq < 4; ++jq)
                    *(lds_u32x2_ptr)(uintptr_t)(ep + e32 * kEpRow + (nb * 32 + 8 * jq + 4 * eh) * 2) =
                        u32x2{f32x2_to_bf16x2(a[4 * jq] + bb, a[4 * jq + 1] + bb), f32x2_to_bf16x2(a[4 * jq + 2] + bb, a[4 * jq + 3] + bb)};
            }
            // (the wave reads what it wrote itself: LDS serves a wave's requests in order)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const int row = it * RPI + el / LPR, m = m0 + mi * 32 + row;
                const uint32_t off = (px_ok & (m < p.M)) ? ((uint32_t)(n * p.M + m) * plane_out + px) * 2u : kNoLoad;
                const uint32_t src = ep + row * kEpRow + seg * (EPI * 2);
                if constexpr (EPI == 8) __builtin_amdgcn_raw_buffer_store_b128(lds16(src), rs_out, off, 0, 0);
                else if constexpr (EPI == 4) __builtin_amdgcn_raw_buffer_store_b64(*(lds_u32x2_ptr)(uintptr_t)src, rs_out, off, 0, 0);
                else if constexpr (EPI == 2) __builtin_amdgcn_raw_buffer_store_b32(*(lds_u32_ptr)(uintptr_t)src, rs_out, off, 0, 0);
                else __builtin_amdgcn_raw_buffer_store_b16(*(lds_u16_ptr)(uintptr_t)src, rs_out, off, 0, 0);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

// ---- few pixels: every wave its own tile, the channels of a tile shared by KS waves
// On small maps the kernel above has a workgroup or less for a compute unit, four waves that wait for the same loads and
// barriers (2048 -> 512 at 7 x 7, batch 64: 128 workgroups of 32 stages in a row, 37 us, matrix pipe 6 % busy).  Here a wave
// owns 64 output channels x 64 pixels and stages them for itself: its 64 lanes are the 64 items of a stage (8 along the
// pixels, 8 along the channels), its part of LDS is its own, and no barrier stands between two stages, so that the eight or
// twelve waves of a compute unit are at different points and fill each other's gaps.  Items of a tile follow one another
// from image to image.  KS waves take every KS-th stage of one tile and add their sums through LDS, in wave order.
// EPI = 16, planes of an odd size up to 56, KS > 1: a tile is whole images, whose 64 channels are one run of memory each, and
// the result leaves in 16-byte stores of that run instead of element by element.
constexpr int kWt = 64, kWtItems = 8;                            // pixels of a wave's tile; items along them
constexpr int kWtBytes = kWt * KCS * 2 + kWtItems * 16;         // a wave's staging buffer
constexpr int kBlk = 64 * 16 * 4;                                // the sums of one 32 x 32 block
constexpr int kWtRow = 32 * 2 + 16;                              // epilogue: a channel's 32 pixels
constexpr int wt_lds(int KS)
{
    const int red = KS > 1 ? 4 * (KS - 1) * (4 / KS) * kBlk : 0;
    return red > 4 * kWtBytes ? red : 4 * kWtBytes;
}

template <int KS, int GW, int EPI, bool TAIL> __global__ void __launch_bounds__(256, 3) conv_pw_wave_kernel(GatherParams p)
{
    constexpr int PT = 4 / KS, KEEP = 4 / KS; // pixel tiles of a workgroup; blocks of 32 x 32 that a wave finishes
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave % KS, pt = wave / KS;
    // every XCD works on consecutive pixel tiles, all output channels of one after the other: its L2 keeps the pixels
    unsigned bx = blockIdx.x, by = 0, bz = 0;
    if constexpr (TAIL) {
        if (!conv_block(p, smem, bx, by, bz)) return;
    }
    const int per_xcd = p.gx >> 3, v = (bx & 7) * per_xcd + (bx >> 3), mtiles = p.Mp / 64;
    if (v >= p.tiles_per_img * mtiles) return; // (tiles_per_img: groups of PT pixel tiles)
    const int grp = v / mtiles, m0 = (v - grp * mtiles) * 64;
    const int ppi = p.Hc * p.Wc, K = p.KCin, nkb = p.nkb, nitems = p.N * p.GX;
    constexpr bool RUNS = EPI == 16;
    const int f0 = (grp * PT + pt) * (RUNS ? p.IPT * p.GX : kWtItems); // the tile's first item

    const int gidx = lane & 7, oct = lane >> 3;
    const int n_it = fdiv(f0 + gidx, p.m_gx);
    const bool item = f0 + gidx < nitems && (!RUNS || gidx < p.IPT * p.GX);
    const uint32_t e0 = item ? (uint32_t)(n_it * K + oct * 8) * ppi + (f0 + gidx - n_it * p.GX) * GW : kNoElem;
    auto pad_of = [](int px) { return GW == 8 ? (px >> 3) * 16 : 0; };
    const uint32_t wbase = lds0 + wave * kWtBytes, l0 = wbase + (uint32_t)(gidx * GW * KCS + oct * 8) * 2u + pad_of(gidx * GW);
    const rsrc_t rs_in = make_rsrc(p.in, (uint32_t)p.N * K * ppi * 2u);
    u32x4 r[8];
    auto fetch = [&](int s) {
        uint32_t e = e0 + (uint32_t)(s * KC) * ppi;
        opaque(e);
        const int nvalid = s < nkb ? K - (s * KC + oct * 8) : 0; // channels that exist
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t ei = i < nvalid ? e : kNoElem;
            r[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, (GW == 7 ? ei & ~1u : ei) * 2u, 0, 0);
            e += ppi;
        }
    };
    auto put = [&](int s) {
        if constexpr (GW == 7) {
            const uint32_t par = e0 + (uint32_t)(s * KC) * ppi;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t sh = ((par + i * ppi) & 1u) * 16u;
#pragma unroll
                for (int k = 0; k < 3; ++k) r[i][k] = __builtin_amdgcn_alignbit(r[i][k + 1], r[i][k], sh);
                r[i][3] >>= sh;
            }
        }
#pragma unroll
        for (int px = 0; px < GW; ++px) {
            u32x4 x; // pixel px of the 8 channels
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t lo = r[2 * k][px / 2], hi = r[2 * k + 1][px / 2];
                x[k] = (px & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
            }
            *(lds_u32x4_ptr)(uintptr_t)(l0 + px * (KCS * 2)) = x;
        }
    };
    // (a wave reads what it wrote itself: LDS serves a wave's requests in order)
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    uint32_t pbase[2];
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) pbase[ni] = wbase + 16u * half + (uint32_t)((ni * 32 + l32) * KCS * 2 + pad_of(ni * 32 + l32));
    const rsrc_t rs_w = make_rsrc(p.wt, p.w_bytes);
    uint32_t wlane[2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
        wlane[mi] = p.w_direct ? (m0 + mi * 32 + l32 < p.M ? (uint32_t)((m0 + mi * 32 + l32) * K + 8 * half) * 2u : kNoLoad)
                               : (uint32_t)((m0 >> 5) + mi) * kFrag + lane * 16u;
    const int ksteps_all = p.KCp / 16;
    u32x4 w[KSTEPS][2];
    auto fetch_w = [&](int s, int kk) {
        const int step = s * KSTEPS + kk; // (16-channel steps past the last one: zeros)
        const uint32_t so = (uint32_t)min(step, ksteps_all - 1) * p.w_kstep;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) w[kk][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, step < ksteps_all ? wlane[mi] : kNoLoad, so, 0);
    };
    f32x16 acc[4]; // block mi + 2 * ni
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[b][j] = 0.f;

    fetch(ks);
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) fetch_w(ks, kk);
    for (int s = ks; s < nkb; s += KS) {
        put(s);
        wave_sync();
        fetch(s + KS); // (past the end: nothing is loaded)
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            union { u32x4 u; bf16x8 v; } a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                b[i].u = lds16(pbase[i] + 32 * kk);
                a[i].u = w[kk][i];
            }
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) acc[2 * ni + mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[ni].v, a[mi].v, acc[2 * ni + mi], 0, 0, 0);
            fetch_w(s + KS, kk);
        }
        wave_sync();
    }
    // ---- the sums of the KS waves: wave ks finishes blocks [ks * KEEP, (ks + 1) * KEEP) and is handed the others' parts of
    // them, red[tile][finishing wave][source wave, itself left out][block]
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    typedef __attribute__((address_space(3))) f32x4 *lds_f32x4_ptr;
    const uint32_t red = lds0 + pt * (KS * (KS - 1) * KEEP * kBlk);
    f32x16 sum[KEEP];
    if constexpr (KS > 1) {
        __syncthreads(); // (all staging buffers are dead)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int dst = b / KEEP;
            if (dst == ks) continue;
            const uint32_t a = red + (uint32_t)(((dst * (KS - 1) + (ks < dst ? ks : ks - 1)) * KEEP + b % KEEP) * kBlk) + lane * 16;
#pragma unroll
            for (int jq = 0; jq < 4; ++jq)
                *(lds_f32x4_ptr)(uintptr_t)(a + jq * 1024) = f32x4{acc[b][4 * jq], acc[b][4 * jq + 1], acc[b][4 * jq + 2], acc[b][4 * jq + 3]};
        }
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < KEEP; ++kb) {
            f32x16 own = acc[kb];
#pragma unroll
            for (int d = 1; d < KS; ++d)
                if (d == ks) own = acc[d * KEEP + kb];
#pragma unroll
            for (int src = 0; src < KS; ++src) {
                f32x16 t = own;
                if (src != ks) {
                    const uint32_t a = red + (uint32_t)(((ks * (KS - 1) + (src < ks ? src : src - 1)) * KEEP + kb) * kBlk) + lane * 16;
#pragma unroll
                    for (int jq = 0; jq < 4; ++jq) {
                        const f32x4 q = *(lds_f32x4_ptr)(uintptr_t)(a + jq * 1024);
#pragma unroll
                        for (int e = 0; e < 4; ++e) t[4 * jq + e] = q[e];
                    }
                }
                if (src == 0) sum[kb] = t;
                else sum[kb] += t;
            }
        }
        wave_sync();
    } else {
#pragma unroll
        for (int b = 0; b < 4; ++b) sum[b % KEEP] = acc[b];
    }
    // ---- epilogue: bias, bfloat16, [channel][pixel] rows in a part of LDS that only this wave uses (KS > 1: what it was handed)
    const rsrc_t rs_out = make_rsrc(p.out, (uint32_t)p.N * p.M * ppi * 2u);
    if constexpr (RUNS) { // [image][channel][pixel] of the whole tile, by the KS waves together
        const uint32_t run = lds0 + pt * (64 * kWtItems * GW * 2);
        __syncthreads(); // (what the others were handed, and read, lies there)
#pragma unroll
        for (int kb = 0; kb < KEEP; ++kb) {
            const int b = ks * KEEP + kb, mi = b & 1, ni = b >> 1, m = m0 + mi * 32 + l32;
            const float bias = (p.bias && m < p.M) ? bf16_to_f32(p.bias[m]) : 0.f;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int idx = ni * 32 + 8 * (j / 4) + 4 * half + j % 4, it = idx / GW;
                const int g = fdiv(it, p.m_gx), px = (it - g * p.GX) * GW + idx - it * GW;
                if ((g < p.IPT) & (px < ppi))
                    *(lds_u16_ptr)(uintptr_t)(run + (uint32_t)((g * 64 + mi * 32 + l32) * ppi + px) * 2u) = f32_to_bf16(sum[kb][j] + bias);
            }
        }
        __syncthreads();
        const int n0 = (grp * PT + pt) * p.IPT, pieces = 8 * ppi, have = min(64, p.M - m0) * ppi / 8; // 16-byte pieces of an image; of them inside
        for (int q = lane + 64 * ks; q < p.IPT * pieces; q += 64 * KS) {
            const int g = fdiv(q, p.m_w2), o = q - g * pieces;
            const uint32_t off = ((n0 + g < p.N) & (o < have)) ? (uint32_t)((n0 + g) * p.M + m0) * ppi * 2u + o * 16u : kNoLoad;
            __builtin_amdgcn_raw_buffer_store_b128(lds16(run + (uint32_t)q * 16u), rs_out, off, 0, 0);
        }
        return;
    }
    const uint32_t ep = KS > 1 ? red + (uint32_t)(ks * (KS - 1) * KEEP * kBlk) : wbase;
    constexpr int LPR = 32 / (RUNS ? 1 : EPI), RPI = 64 / LPR; // lanes of a row; rows per pass over the lanes
#pragma unroll
    for (int kb = 0; kb < KEEP; ++kb) {
        const int b = ks * KEEP + kb, mi = b & 1, ni = b >> 1;
        const int mb = m0 + mi * 32;
        const float bias = (p.bias && mb + l32 < p.M) ? bf16_to_f32(p.bias[mb + l32]) : 0.f;
#pragma unroll
        for (int jq = 0; jq < 4; ++jq)
            *(lds_u32x2_ptr)(uintptr_t)(ep + l32 * kWtRow + (8 * jq + 4 * half) * 2) =
                u32x2{f32x2_to_bf16x2(sum[kb][4 * jq] + bias, sum[kb][4 * jq + 1] + bias), f32x2_to_bf16x2(sum[kb][4 * jq + 2] + bias, sum[kb][4 * jq + 3] + bias)};
        wave_sync();
        const int seg = lane % LPR, idx = ni * 32 + seg * EPI, it = idx / GW;
        const int n = fdiv(f0 + it, p.m_gx), px = (f0 + it - n * p.GX) * GW + idx - it * GW;
        const bool ok = (it < kWtItems) & (f0 + it < nitems) & (px < ppi);
#pragma unroll
        for (int t = 0; t < 32 / RPI; ++t) {
            const int row = t * RPI + lane / LPR, m = mb + row;
            const uint32_t off = (ok & (m < p.M)) ? ((uint32_t)(n * p.M + m) * ppi + px) * 2u : kNoLoad;
            const uint32_t src = ep + row * kWtRow + seg * (EPI * 2);
            if constexpr (EPI == 8) __builtin_amdgcn_raw_buffer_store_b128(lds16(src), rs_out, off, 0, 0);
            else if constexpr (EPI == 4) __builtin_amdgcn_raw_buffer_store_b64(*(lds_u32x2_ptr)(uintptr_t)src, rs_out, off, 0, 0);
            else if constexpr (EPI == 2) __builtin_amdgcn_raw_buffer_store_b32(*(lds_u32_ptr)(uintptr_t)src, rs_out, off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b16(*(lds_u16_ptr)(uintptr_t)src, rs_out, off, 0, 0);
        }
        wave_sync();
    }
}

template <int KS, int GW, int EPI, bool TAIL> hipError_t launch_wave_kernel(const GatherParams &p, hipStream_t st)
{
    auto kern = conv_pw_wave_kernel<KS, GW, EPI, TAIL>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    const int total = p.tiles_per_img * (p.Mp / 64);
    GatherParams q = p;
    const dim3 grid = share_grid(q, dim3((total + 7) / 8 * 8), 256);
    hipLaunchKernelGGL(kern, grid, dim3(256), wt_lds(KS), st, q);
    return hipGetLastError();
}
template <int KS, int GW, int EPI> hipError_t launch_wave_fixed(const GatherParams &p, hipStream_t st)
{
    return p.tail.blocks ? launch_wave_kernel<KS, GW, EPI, true>(p, st) : launch_wave_kernel<KS, GW, EPI, false>(p, st);
}
template <int KS> hipError_t launch_wave(const GatherParams &p, hipStream_t st)
{
    if constexpr (KS > 1)
        if (p.store_px == 16) return launch_wave_fixed<KS, 7, 16>(p, st);
    if (p.gw == 7) return launch_wave_fixed<KS, 7, 1>(p, st);
    return p.store_px == 8 ? launch_wave_fixed<KS, 8, 8>(p, st) : p.store_px == 4 ? launch_wave_fixed<KS, 8, 4>(p, st)
                                                                                  : launch_wave_fixed<KS, 8, 2>(p, st);
}

template <int NI, int WM, int WN, bool FUSE, int GW, int EPI, bool TAIL> hipError_t launch_kernel(const GatherParams &p, hipStream_t st)
{
    auto kern = conv_pw_kernel<NI, WM, WN, FUSE, GW, EPI, TAIL>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    dim3 grid(p.tiles_per_img * p.ngrp, (p.Mp / 64 + WM - 1) / WM);
    GatherParams q = p;
    grid = share_grid(q, grid, 256);
    hipLaunchKernelGGL(kern, grid, dim3(256), 2 * kBuf, st, q);
    return hipGetLastError();
}
template <int NI, int WM, int WN, bool FUSE, int GW, int EPI> hipError_t launch_fixed(const GatherParams &p, hipStream_t st)
{
    if constexpr (!FUSE) // (a forward pass)
        if (p.tail.blocks) return launch_kernel<NI, WM, WN, FUSE, GW, EPI, true>(p, st);
    return launch_kernel<NI, WM, WN, FUSE, GW, EPI, false>(p, st);
}
template <int NI, int WM, int WN> hipError_t launch_shape(const GatherParams &p, hipStream_t st)
{
    if (p.Z) return launch_fixed<NI, WM, WN, true, 8, 8>(p, st); // (rows of a multiple of 4, an even number of them)
    if (p.gw == 7) return launch_fixed<NI, WM, WN, false, 7, 1>(p, st);
    return p.store_px == 8 ? launch_fixed<NI, WM, WN, false, 8, 8>(p, st) : p.store_px == 4 ? launch_fixed<NI, WM, WN, false, 8, 4>(p, st)
                                                                                  : launch_fixed<NI, WM, WN, false, 8, 2>(p, st);
}
struct Shape { int ni, wm, wn; hipError_t (*launch)(const GatherParams &, hipStream_t); };
const Shape kShapes[] = {{2, 1, 4, launch_shape<2, 1, 4>}, {4, 2, 2, launch_shape<4, 2, 2>}};
constexpr int kWaveVariant = 2; // from here on: conv_pw_wave_kernel with KS = 1 and 4
hipError_t (*const kWaves[])(const GatherParams &, hipStream_t) = {launch_wave<1>, launch_wave<4>};
int waves_of(int variant) { return variant == kWaveVariant ? 1 : 4; }

} // namespace

// Plans a 1 x 1 stride-1 launch (p: N, M, Mp, KCin, Hin, Win, Hc, Wc filled in); false when it is not its own.
// pool: the 2 x 2 mean record of the input is wanted (p.pw_pool tells whether the launch forms it); record_free: the
// launches of conv_mfma.hip would form it in their repack.  *gather: those launches, where they take the layer, measured
// the faster ones; *gather_whole: where they also need no finishing launch.
bool shape_pw(GatherParams &p, bool pool, bool record_free, int *variant, bool *gather, bool *gather_whole)
{
    if (p.ntaps != 1 || p.os != 1 || p.is != 1 || p.decim || p.dh[0] || p.dw[0] || p.Hin != p.Hc || p.Win != p.Wc) return false;
    GatherParams q = p;
    const int ppi = p.Hc * p.Wc;
    q.KCp = (p.KCin + 15) / 16 * 16;
    q.nkb = q.kbs = (p.KCin + KC - 1) / KC;
    q.ksplit = 1; q.gpw = 1; q.part = nullptr; q.T = 1;
    q.gw = ppi % 2 ? 7 : 8;
    q.store_px = ppi % 8 == 0 ? 8 : ppi % 4 == 0 ? 4 : ppi % 2 == 0 ? 2 : 1;
    q.pw_pool = pool && p.Win % 4 == 0 && p.Hin % 2 == 0 && p.Win / 4 <= kGroups && ppi >= kPT / 2 && 2L * ppi * p.Win < 1L << 32;
    // Up to 32 channels leave half of the threads or more without an item, and the others would pool as well as stage: on
    // maps that fill the chip a compress launch is the cheaper way (10 -> 14 at 68 x 68, batch 198: 72 -> 40 us).
    if (p.KCin <= 32 && (long)p.N * ppi >= 512L * kPT) q.pw_pool = 0;
    if (q.pw_pool) {
        q.GX = p.Win / 4;
        q.IPT = 1;
        q.tile_px = min(kGroups / q.GX, p.Hin / 2) * 2 * p.Win;
    } else {
        const int gi = (ppi + q.gw - 1) / q.gw; // items along a plane
        q.IPT = 2 * gi <= kGroups ? min(kGroups / gi, p.N) : 1;
        q.GX = gi;
        q.tile_px = q.IPT > 1 ? ppi : kGroups * q.gw;
    }
    q.tiles_per_img = q.IPT > 1 ? 1 : (ppi + q.tile_px - 1) / q.tile_px;
    q.ngrp = (p.N + q.IPT - 1) / q.IPT;
    q.m_gx = magic_of(q.GX); q.m_ppi = magic_of(q.GX * q.gw); q.m_w2 = magic_of(2 * p.Win);
    const long px_tiles = (long)q.tiles_per_img * q.ngrp;
    if (px_tiles > 0x7fffffffL) return false;
    // 128 output channels per workgroup where that still gives every compute unit a workgroup: half the input traffic
    // (64 -> 256 at 56 x 56, batch 64: 39 against 50 us; 256 -> 1024 at 14 x 14 backwards, 128 workgroups: 29 against 23).
    int v = q.Mp > 64 && px_tiles * ((q.Mp + 127) / 128) >= 256;
#ifdef CAC_TUNING
    if (const char *f = getenv("CAC_PW_SHAPE")) v = atoi(f);
#endif
    const long wgs = px_tiles * ((q.Mp / 64 + kShapes[v].wm - 1) / kShapes[v].wm);
    // Fragments from W itself touch 32 lines each, repacked ones 8, but save the repack launch: faster on small inputs
    // (256 -> 64 at 56 x 56, batch 2: 12.2 against 14.2 us) and while a workgroup of 128 channels has few stages
    // (512 -> 128 at 28 x 28, 2048 of them: 28.6 against 29.9 us; 384 -> 359 at 9 x 33, batch 139, 5000: 65 against 59).
    q.w_direct = v == 1 ? wgs * q.nkb <= 2560 : q.nkb <= 2 || (q.nkb <= 8 && wgs * q.nkb <= 256);
    // A handful of workgroups with a long sum each: the launches of conv_mfma.hip share out the channels (512 -> 128 at
    // 28 x 28, batch 4, 32 workgroups of 8 stages: 18.8 against 20.1 us; 2048 -> 512 at 7 x 7, batch 8: 36 against 42).
    *gather = wgs < 64 && q.nkb >= 8;
    // Planes of two or four pixels fill half of a tile's items at most (512 -> 1024 at 2 x 2, batch 1500, data gradient: 22
    // against 45 us).  Single pixels a seventh, but those the gather copies one by one (1024 -> 1024, batch 2048: 134
    // against 66 us).
    *gather |= ppi <= 4 && ppi % 2 == 0 && wgs >= 64 && q.nkb >= 4;
    // The same for more of them, or for shorter sums, where the stages pool, and every tile of output channels pools anew
    // (1299 -> 1095 at 12 x 12, batch 8, 144 workgroups: 28.9 against 54.2 us; 803 -> 73 at 16 x 16, batch 32, 64 of them:
    // 18.6 against 32.0).  Of random layers those within the lines ran at 1.1-1.65 of the gather's time in the mean, those
    // just past them at 0.75-1.04.  Fewer than eight stages only if rows of W are not whole items: the filter's repack, a
    // launch of its own here, then takes longer (250 -> 16 at 16 x 16, batch 6: 14.4 against 13.3 us; but 256 -> 64 at
    // 56 x 56, batch 2: 11.7 against 15.8; 256 -> 128, batch 4, which repacks too: 14.2 against 16.2).
    if (q.pw_pool && (q.nkb >= 8 || (q.nkb >= 4 && q.KCin % 8))) {
        const bool one = wgs == px_tiles; // one tile of output channels
        *gather |= one ? wgs < (q.nkb >= 16 ? 128 : q.nkb >= 8 || record_free ? 64 : 0)
                       : wgs < (q.nkb >= 8 ? 256 : record_free ? 128 : 64);
    }
    // For any length where the record would need a launch of its own here that the gather's repack saves (45 -> 20 at 8 x 8,
    // batch 168: 10.4 against 13.1 us; 1.2 of its time in the mean, 0.83 from 256 workgroups on), unless the gather shares
    // out its channels, which is a launch more as well (1.0).
    *gather_whole = !q.pw_pool && wgs < 256 && record_free;
    *variant = v;
    // By waves, where the items are full (planes of 1 to 4 pixels: as above).  Measured on 2885 random calls against the launches
    // above and the gather's: four waves to a tile take 0.53-0.6 of the time up to 256 tiles of 64 x 64 with eight stages or
    // more (2048 -> 512 at 7 x 7, batch 64: 46.9 -> 28.8 us; the data gradient of 512 -> 2048 43.8 -> 24.4), 0.73-1.0 up to the line below
    // and 0.8-0.97 with four to seven stages up to theirs, 1.05-1.15 past them (wave tiles are 64 channels wide, and their operands
    // come through L2 once per 64 x 64).  With three stages, or fewer, a hand-over costs what it saves (0.95-1.3), but many
    // tiles of one wave each keep more loads in flight than the shapes above (0.75-0.93).
    const int gx = (ppi + q.gw - 1) / q.gw;
    const long items = (long)p.N * gx;
    bool runs = q.gw == 7 && gx <= kWtItems && q.M % 8 == 0; // tiles of whole images, each a run of whole 16-byte pieces
    const int ipt = runs ? kWtItems / gx : 1;
    long tiles = runs ? (p.N + ipt - 1) / ipt : (items + kWtItems - 1) / kWtItems, wt = tiles * (q.Mp / 64);
    int ks = 0;
    if (q.nkb >= 4 && wt < (q.nkb >= 8 ? 2048 : 1024)) {
        ks = 4;
    } else {
        // One wave hands out a run's elements two bytes at a time between barriers that the workgroup's other tiles wait for, and
        // whole images leave a tile emptier: 1.1 of the time of the shapes above, worst 1.38 (128 -> 1648 at 7 x 7, batch 124: 28.1
        // against 20.5 us), where items that run on take 0.87, worst 1.12 (420 random calls; 0.80 of the time with runs).
        runs = false;
        tiles = (items + kWtItems - 1) / kWtItems;
        wt = tiles * (q.Mp / 64);
        if (q.nkb < 3 ? wt >= 2048 : q.nkb >= 4 && q.nkb < 8 && wt >= 4096) ks = 1;
    }
    // Nor where the shapes above, two workgroups to a compute unit, find the chip just about full -- 385 to 512 of them all start
    // at once -- and little of their tiles is padding: four waves to a tile then take 1.07 of their time with six tiles of output
    // channels or more (0.91 with two to four, whose pixels pass L2 less often), one wave to a tile 1.07 on planes of an even
    // size (0.97 on odd ones); up to 1.28 (816 -> 1824 at 5 x 43, batch 15, 435 workgroups, 30.8 against 39.2 us).  Outside of the
    // window a last round or a half-empty chip costs those shapes more than that.
    if (!*gather && wgs > 384 && wgs <= 512 && 5 * wt >= 16 * wgs * kShapes[v].wm && (ks == 4 ? q.Mp >= 384 : q.gw == 8)) ks = 0;
#ifdef CAC_TUNING
    if (const char *f = getenv("CAC_PW_WAVE")) if (atoi(f) < 0) ks = 0;
#endif
    // Not where the record is pooled on the way, which is worth more than the waves, nor for fewer than eight tiles of a layer
    // that the gather takes: those are too few to matter (1 in 50 random layers; 0.65 of the time) and keep its channel split
    // in use and under test.
    if (ks && !q.pw_pool && (!*gather || wt >= 8) && 2 * ppi > gx * q.gw && divides_exactly((uint64_t)items + kWtItems * 4, gx)) {
        q.GX = gx;
        q.m_gx = magic_of(gx);
        q.IPT = runs ? ipt : 1;
        q.ngrp = 1;
        q.tile_px = kWt;
        const int pt = 4 / ks;
        q.tiles_per_img = (int)((tiles + pt - 1) / pt);
        if (runs) {
            q.store_px = 16;
            q.m_w2 = magic_of(8 * ppi); // (16-byte pieces of an image; a tile has at most 448)
        }
        // fragments from W itself: 0.85-0.95 of the time with a repack launch for four waves to a tile, 1.04 for many tiles with
        // long sums; 0.9-0.98 for one wave to a tile with one or two stages
        q.w_direct = ks == 4 ? wt < 512 || q.nkb < 16 : q.nkb < 3;
        *variant = kWaveVariant + (ks == 4);
        *gather = *gather_whole = false;
    }
    p = q;
    return true;
}

hipError_t launch_pw(const GatherParams &p, int variant, hipStream_t st)
{
    return variant >= kWaveVariant ? kWaves[variant - kWaveVariant](p, st) : kShapes[variant].launch(p, st);
}

int describe_pw(const GatherParams &p, int variant, char *buf, size_t len)
{
    if (variant >= kWaveVariant)
        return snprintf(buf, len, "pointwise by waves tile=64ch x %dpx ch/pass=%d waves/tile=%d grid=%dx1x1 lds=%dB, input read in place", p.store_px == 16 ? p.IPT * p.Hc * p.Wc : kWtItems * p.gw, KC,
                        waves_of(variant), (p.tiles_per_img * (p.Mp / 64) + 7) / 8 * 8, wt_lds(waves_of(variant)));
    const Shape &v = kShapes[variant];
    return snprintf(buf, len, "pointwise tile=%dch x %dpx ch/pass=%d img/tile=%d grid=%dx%dx1 lds=%dB%s, input read in place", 64 * v.wm, p.tile_px, KC, p.IPT,
                    p.tiles_per_img * p.ngrp, (p.Mp / 64 + v.wm - 1) / v.wm, 2 * kBuf, p.pw_pool ? ", pooled on the way" : "");
}

} // namespace cac
