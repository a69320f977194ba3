// Data gradient of a 3 x 3 convolution with stride 2 and padding 1 on maps of even width: one launch for all four
// parity classes of the input pixel.
//
//   dX[n, c, 2i + a0, 2j + b0] = sum_{o, taps of (a0, b0)} W[o][c][r][s] * dY[n, o, i + dh, j + dw]
// with the taps r = 1 (a0 = 0, dh = 0), r = 0 (a0 = 1, dh = 1), r = 2 (a0 = 1, dh = 0), columns likewise: nine
// (class, tap) pairs over four shifts (dh, dw) of one and the same dY patch.  A launch per class (conv_mfma.hip) reads
// and repacks dY four times, has one, two, two and four taps to hide its loads behind and writes every second pixel
// as 2-byte stores.  Here a wave owns 32 channels c x 64 pixels (i, j) of dY x the four classes (128 accumulators);
// per 16 channels o it takes eight pixel fragments from LDS and nine filter fragments from the caches (a ring of
// nine in flight) for eighteen MFMAs, and the classes leave together: the two of a row side by side as dwords,
// through LDS, so that the lanes of a store cover whole output rows.  Staging and the pairing of two workgroups per
// compute unit are those of conv_tile.hip.  Per call, batch 128: 128 -> 256 at 28 x 28 71 -> 31 us, 64 -> 128 at 56 x 56
// 101 -> 35 us, 256 -> 512 at 14 x 14 77 -> 34 us; a batch of 2 of the second 37 -> 13.5 us.
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

// (class, tap, shift = 2 * dh + dw), the shifts in the order 1, 0, 2, 3.  Their pixel fragments live in three register
// sets that rotate from one 16-channel step to the next, each requested as soon as a set is free: six MFMAs or more
// ahead of their use, except for the first ones of a stage.
constexpr int kCls[9] = {1, 3, 0, 1, 2, 3, 2, 3, 3};
constexpr int kTap[9] = {3, 6, 4, 5, 7, 8, 1, 2, 0};
constexpr int kShift[9] = {1, 1, 0, 0, 0, 0, 2, 2, 3};
// set of a shift at step kk: at step 0 shift 0 in set 0, shifts 1 and 3 in set 1, shift 2 in set 2; from step to step
// (0, 1, 2) become (2, 0, 1)
constexpr int set_of(int shift, int kk) { return ((shift == 0 ? 0 : shift == 2 ? 2 : 1) + 2 * kk) % 3; }
constexpr int kNI = 2;                                 // 32-pixel blocks of a wave
constexpr int kEpRow = 64 * 4 + 16;                    // LDS bytes of an epilogue row: 64 pairs of pixels
constexpr int kEpWave = 32 * kEpRow;

// KC: channels o of a stage (32 or 64); EPI: dwords (pairs of output pixels) per store; TAIL: the launch may have workgroups that add
// a weight gradient's slices (a form of its own: where all registers are in use the branch alone costs 2-6 %).
template <int WM, int WN, int ITEMS, int GW, int KC, int EPI, bool TAIL>
__global__ void __launch_bounds__(256, 2) conv_dx2_kernel(GatherParams p)
{
    constexpr int PT = WN * kNI * 32, KS = KC / 16;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint32_t buf_bytes = p.buf_bytes;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;
    unsigned bx = blockIdx.x, by = blockIdx.y, bz = 0;
    if constexpr (TAIL) {
        if (!conv_block(p, smem, bx, by, bz)) return;
    }
    const int tau = bx / p.ngrp, n_base = (bx - tau * p.ngrp) * p.IPT;
    const int nkb = p.nkb, ppi = p.Hc * p.Wc;
    const int pix0 = p.IPT > 1 ? 0 : tau * PT, i0 = fdiv(pix0, p.m_wc);
    const int m0 = (by * WM + wm) * 32;

    PatchStage<ITEMS, GW, KC> in;
    in.init(p, lds0, lds0 + 2 * buf_bytes, n_base, i0);
    constexpr int KCS = KC + 8;

    uint32_t pbase[kNI]; // this lane's pixels (shift (0, 0))
#pragma unroll
    for (int ni = 0; ni < kNI; ++ni) {
        const int idx = (wn * kNI + ni) * 32 + l32;
        int g = 0, px = pix0 + idx;
        bool ok = px < ppi;
        if (p.IPT > 1) {
            g = fdiv(idx, p.m_ppi);
            px = idx - g * ppi;
            ok = g < p.IPT;
        }
        const int i = fdiv(px, p.m_wc), j = px - i * p.Wc;
        pbase[ni] = lds0 + 16u * half + (ok ? (uint32_t)(((g * p.PH + i - i0) * p.PWd + j) * KCS * 2) : 0u);
    }
    const rsrc_t rs_w = make_rsrc(p.wt, 9u * p.Mp * p.KCp * 2u);
    const uint32_t kstep = p.Mp / 32 * kFrag;
    const uint32_t wlane = m0 < p.Mp ? (uint32_t)(m0 >> 5) * kFrag + lane * 16u : kNoLoad;
    const rsrc_t rs_out = make_rsrc(p.out, (uint32_t)p.N * p.M * p.Hout * p.Wout * 2u);
    // pixel blocks of this wave that hold any pixel
    const int nlive = p.IPT > 1 ? kNI : max(0, min(kNI, (ppi - pix0 - wn * kNI * 32 + 31) / 32));

    auto run_wave = [&](auto nltag) {
    constexpr int NL = decltype(nltag)::value, NA = NL > 0 ? NL : 1;
    f32x16 acc[4][NA];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int ni = 0; ni < NA; ++ni)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[c][ni][j] = 0.f;
    u32x4 wr[9]; // filter fragments of the current 16 channels, each replaced by the next 16 channels' once used
#pragma unroll
    for (int t = 0; t < 9; ++t) wr[t] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, p.wofs[kTap[t]], 0);
    in.start(lds0, buf_bytes);

    const int ksteps = p.KCp / 16;
    for (int s = 0; s < nkb; ++s) {
        const uint32_t buf = (s & 1) ? buf_bytes : 0u, nbuf = buf_bytes - buf;
        in.fetch(s + 1, 0); // (past the end: nothing is loaded)
        u32x4 b[3][NA];
        auto ask = [&](int shift, int kk) {
#pragma unroll
            for (int ni = 0; ni < NL; ++ni) b[set_of(shift, kk)][ni] = lds16(pbase[ni] + p.toff[shift] + 32 * kk);
        };
        ask(1, 0);
        ask(0, 0);
        ask(2, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            uint32_t so = (uint32_t)min(s * KS + kk + 1, ksteps - 1) * kstep; // (after the last step: read again, never used)
            opaque_s(so);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                if constexpr (NL > 0) {
#pragma unroll
                    for (int ni = 0; ni < NL; ++ni) {
                        union { u32x4 u; bf16x8 v; } af, bf;
                        af.u = wr[t];
                        bf.u = b[set_of(kShift[t], kk)][ni];
                        acc[kCls[t]][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf.v, af.v, acc[kCls[t]][ni], 0, 0, 0);
                    }
                    wr[t] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, p.wofs[kTap[t]] + so, 0);
                    if (t == 1) ask(3, kk);
                    if (kk + 1 < KS) {
                        if (t == 5) ask(1, kk + 1);
                        if (t == 7) ask(0, kk + 1);
                        if (t == 8) ask(2, kk + 1);
                    }
                }
                // staging: two halves per stage, loads at the first of W steps, the pixels to LDS at the last eight
                constexpr int W = 9 * KS / 2;
                const int q = kk * 9 + t, h = q / W, qq = q - h * W;
                if (qq == W - 9) in.align_rows();
                if (qq >= W - 8) in.put_px(nbuf, h, qq - (W - 8));
                if (qq == W - 1 && h == 0) in.fetch(s + 1, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // on to the other buffer
#pragma unroll
        for (int ni = 0; ni < NL; ++ni) {
            pbase[ni] += nbuf - buf;
            opaque(pbase[ni]);
        }
        __syncthreads();
    }
    // ---- epilogue: the two classes of an output row side by side, 32 channels x 64 pairs at a time through LDS (the
    // staging buffers are dead), every wave in a part of its own
    const uint32_t ep = lds0 + wave * kEpWave;
    uint32_t el = lane;
    opaque(el);
    const uint32_t eh = el >> 5, e32 = el & 31;
    constexpr int LPR = NA * 32 / EPI, RPI = 64 / LPR; // lanes of a row; rows per pass over the lanes
    const int seg = el % LPR, idx = wn * kNI * 32 + seg * EPI;
    int g = 0, px = pix0 + idx;
    if (p.IPT > 1) {
        g = fdiv(idx, p.m_ppi);
        px = idx - g * ppi;
    }
    const int n = n_base + g, i = fdiv(px, p.m_wc), j = px - i * p.Wc;
    const bool px_ok = (px < ppi) & (g < p.IPT) & (n < p.N) & (NL > 0);
#pragma unroll
    for (int a0 = 0; a0 < 2; ++a0) {
#pragma unroll
        for (int nb = 0; nb < NL; ++nb) {
            const f32x16 &l = acc[2 * a0][nb], &r = acc[2 * a0 + 1][nb];
#pragma unroll
            for (int jq = 0; jq < 4; ++jq)
                *(lds_u32x4_ptr)(uintptr_t)(ep + e32 * kEpRow + (nb * 32 + 8 * jq + 4 * eh) * 4) =
                    u32x4{f32x2_to_bf16x2(l[4 * jq], r[4 * jq]), f32x2_to_bf16x2(l[4 * jq + 1], r[4 * jq + 1]),
                          f32x2_to_bf16x2(l[4 * jq + 2], r[4 * jq + 2]), f32x2_to_bf16x2(l[4 * jq + 3], r[4 * jq + 3])};
        }
        // (the wave reads what it wrote itself: LDS serves a wave's requests in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const bool ok = px_ok & (2 * i + a0 < p.Hout);
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int row = it * RPI + el / LPR, m = m0 + row;
            const uint32_t off = (ok & (m < p.M)) ? (((uint32_t)(n * p.M + m) * p.Hout + 2 * i + a0) * p.Wout + 2 * j) * 2u : kNoLoad;
            const uint32_t src = ep + row * kEpRow + seg * (EPI * 4);
            if constexpr (EPI == 4) __builtin_amdgcn_raw_buffer_store_b128(lds16(src), rs_out, off, 0, 0);
            else if constexpr (EPI == 2) __builtin_amdgcn_raw_buffer_store_b64(*(lds_u32x2_ptr)(uintptr_t)src, rs_out, off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b32(*(lds_u32_ptr)(uintptr_t)src, rs_out, off, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    };
    if (nlive == 2) run_wave(std::integral_constant<int, 2>{});
    else if (nlive == 1) run_wave(std::integral_constant<int, 1>{});
    else run_wave(std::integral_constant<int, 0>{});
}

template <int WM, int WN, int ITEMS, int GW, int KC, int EPI, bool TAIL> hipError_t launch_kernel(const GatherParams &p, hipStream_t st)
{
    auto kern = conv_dx2_kernel<WM, WN, ITEMS, GW, KC, EPI, TAIL>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    dim3 grid(p.tiles_per_img * p.ngrp, (p.Mp / 32 + WM - 1) / WM);
    GatherParams q = p;
    grid = share_grid(q, grid, 256);
    hipLaunchKernelGGL(kern, grid, dim3(256), p.lds_bytes, st, q);
    return hipGetLastError();
}
template <int WM, int WN, int ITEMS, int GW, int KC, int EPI> hipError_t launch_fixed(const GatherParams &p, hipStream_t st)
{
    return p.tail.blocks ? launch_kernel<WM, WN, ITEMS, GW, KC, EPI, true>(p, st) : launch_kernel<WM, WN, ITEMS, GW, KC, EPI, false>(p, st);
}
template <int WM, int WN, int ITEMS, int KC> hipError_t launch_rows(const GatherParams &p, hipStream_t st)
{
    if (p.gw == 7) return launch_fixed<WM, WN, ITEMS, 7, KC, 1>(p, st); // rows of odd length
    return p.store_px == 4 ? launch_fixed<WM, WN, ITEMS, 8, KC, 4>(p, st) : launch_fixed<WM, WN, ITEMS, 8, KC, 2>(p, st);
}
template <int WM, int WN> hipError_t launch_shape(const GatherParams &p, hipStream_t st)
{
    if (p.T == 2) return launch_rows<WM, WN, 1, 64>(p, st); // (never planned with two items per thread)
    const bool one = p.IPT * p.PH * p.GX * 4 <= 256;
    return one ? launch_rows<WM, WN, 1, 32>(p, st) : launch_rows<WM, WN, 2, 32>(p, st);
}

struct Shape { int wm, wn; hipError_t (*launch)(const GatherParams &, hipStream_t); };
const Shape kShapes[] = {{1, 4, launch_shape<1, 4>}, {2, 2, launch_shape<2, 2>}};

} // namespace

// Plans the launch; false when the geometry is not its own.  p: N, M (= C_in), Mp, KCin (= C_out), Hin, Win (of dY),
// Hout, Wout (of dX) are filled in.
bool shape_dx2(const Geom &g, GatherParams &p, int *variant, double *cost_out)
{
    if (g.R != 3 || g.S != 3 || g.sh != 2 || g.sw != 2 || g.ph != 1 || g.pw != 1 || g.W % 2) return false;
    GatherParams b = p;
    b.Hc = g.P; b.Wc = g.Q; // (H odd or even: ceil(H / 2) rows of every class, the second one's last may not exist)
    b.dhmin = b.dwmin = 0;
    b.PWd = g.Q + 1;
    b.os = 2; b.is = 1; b.ntaps = b.ntaps_total = 9;
    b.ksplit = 1; b.gpw = 1; b.part = nullptr;
    const int ppi = g.P * g.Q;
    if (!divides_exactly(ppi, g.Q)) return false; // (a pixel's row and column)
    b.gw = g.Q % 2 ? 7 : 8;
    b.GX = (g.Q + b.gw - 1) / b.gw;
    b.store_px = g.Q % 4 == 0 ? 4 : g.Q % 2 == 0 ? 2 : 1;
    b.m_wc = magic_of(g.Q); b.m_ppi = magic_of(ppi); b.m_gx = magic_of(b.GX);
    GatherParams best{};
    double best_cost = 1e300;
    int f = -1;
#ifdef CAC_TUNING
    if (const char *force = getenv("CAC_DX2_SHAPE")) f = atoi(force); // 2 * shape + (64 channels per stage)
#endif
    for (int v = 0; v < (int)(sizeof(kShapes) / sizeof(kShapes[0])); ++v)
        for (int t : {2, 1}) {
            if (f >= 0 && f != 2 * v + (t == 2)) continue;
            const Shape &sh = kShapes[v];
            if (t == 2 && b.KCin <= 32) continue;
            if (sh.wm * 32 > b.Mp) continue;
            GatherParams q = b;
            const int kc = 32 * t, pt = sh.wn * kNI * 32, kcs = kc + 8;
            q.T = t;
            q.KCp = (b.KCin + kc - 1) / kc * kc;
            q.nkb = q.kbs = q.KCp / kc;
            q.IPT = 2 * ppi <= pt ? min(pt / ppi, g.N) : 1;
            q.tiles_per_img = q.IPT > 1 ? 1 : (ppi + pt - 1) / pt;
            q.PH = (q.IPT > 1 ? g.P : min(g.P, (pt + g.Q - 2) / g.Q + 1)) + 1;
            const int items = q.IPT * q.PH * q.GX * (kc / 8);
            if (items > (t == 2 ? 256 : 512)) continue; // (64 channels in two items per thread: 32 in one are always the cheaper)
            q.patch_px = q.IPT * q.PH * q.PWd;
            q.buf_bytes = max(q.patch_px * kcs * 2, 2 * kEpWave);
            q.lds_bytes = 2 * q.buf_bytes + kDumpBytes;
            if (q.lds_bytes > 160 * 1024) continue;
            q.m_ph = magic_of(q.PH);
            q.ngrp = (g.N + q.IPT - 1) / q.IPT;
            const uint32_t mblks = q.Mp / 32;
            for (int tap = 0; tap < 9; ++tap) q.wofs[tap] = (uint32_t)tap * (q.KCp / 16) * mblks * kFrag;
            for (int s = 0; s < 4; ++s) q.toff[s] = (uint32_t)((s >> 1) * q.PWd + (s & 1)) * kcs * 2u;
            const long wgs = (long)q.tiles_per_img * q.ngrp * ((mblks + sh.wm - 1) / sh.wm);
            // rough cycles of a compute unit: the MFMAs at half rate, a barrier per stage, a start and an epilogue
            const bool pairs = wgs > 256 && q.lds_bytes <= 80 * 1024;
            const double k = (double)((wgs + 255) / 256);
            // (128 accumulators, nine filter and six pixel fragments leave too little of 256 registers for the staging: one item
            // per thread spills 4 to 15 of them, two up to 40)
            const double spilled = items <= 256 ? 1.0 : 1.2;
            const double cost = k * q.nkb * spilled * (18.0 * 32 * 2 * t / (pairs ? 0.5 : 0.35) + (pairs ? 300 : 600)) + (pairs ? (k + 1) / 2 : k) * 8000.0;
            if (cost < best_cost) {
                best_cost = cost;
                best = q;
                *variant = v;
            }
        }
    if (best_cost > 1e299) return false;
    p = best;
    *cost_out = best_cost;
    return true;
}

hipError_t launch_dx2(const GatherParams &p, int variant, hipStream_t st) { return kShapes[variant].launch(p, st); }

int describe_dx2(const GatherParams &p, int variant, char *buf, size_t len)
{
    const Shape &v = kShapes[variant];
    return snprintf(buf, len, "tile=%dch x 4 x %dpx (four parity classes, WM=%d WN=%d) taps=9 ch/pass=%d img/tile=%d patch=%dx%d grid=%dx%dx1 lds=%dB",
                    32 * v.wm, kNI * 32 * v.wn, v.wm, v.wn, 32 * p.T, p.IPT, p.PH, p.PWd, p.tiles_per_img * p.ngrp, (p.Mp / 32 + v.wm - 1) / v.wm,
                    p.lds_bytes);
}

} // namespace cac
