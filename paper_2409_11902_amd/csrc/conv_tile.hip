// Nine-tap gather GEMM (3 x 3 forward convolution, stride 1 or 2, and 3 x 3 stride-1 data gradient) with large
// wave tiles.
//
// The sum is the one of conv_mfma.hip, filter fragments and taps as there.  What bounds that file's kernel on
// layers with enough pixels is the vector cache: its four MFMA waves of 64 channels x 64 pixels ask it for
// 64 bytes of filter fragments per clock, its peak, and half of the register file belongs to copy waves.  Here
//   - a workgroup is four waves that all do the same, stage and multiply, and two workgroups share a compute
//     unit (256 registers a wave): what one waits for -- a barrier, the input of its next stage, its epilogue --
//     the other fills;
//   - a wave owns 64 output channels x 128 (or 64) pixels, so that a filter fragment serves four (two) MFMAs
//     and a pixel fragment two: 32 bytes per clock from the vector cache and 64 from LDS, half of either's peak;
//   - the input is read where it lies ([N][C][H][W], rows of any length): every thread moves items of 8
//     channels x 8 pixels (7 in rows of odd length) in two halves of 4 channels through 16 registers, loads at
//     the first of nine steps, an in-register transpose and the LDS writes between the MFMAs of the last four;
//   - pixel blocks of an image's last tile that hold no pixel are not multiplied (a wave runs the loop compiled
//     for the number of blocks it has).
// Measured per call (repack launch included; bench layers): 512 -> 512 at 14 x 14, batch 256, data gradient
// 325 -> 210-240 us (1.0-1.1 PFLOP/s of useful work; the chip is power-limited here: 1.8 GHz at 70 % MFMA
// utilisation, a large library matrix product reaches 1.29 PFLOP/s on the same box); 512 -> 512 at 7 x 7
// 98 -> 71 us; 128 -> 128 at 28 x 28, batch 128, 51 -> 36 us; 64 -> 64 at 56 x 56, batch 64, 43 -> 28 us.
// Eight steps of filter fragments in flight instead of three, or a whole stage fetched at once through 32
// registers, measured the same or slower; 64 x 224 pixels per wave with 512 registers does not fit (spills).  Two 7-pixel
// items per thread spill 10 to 15 registers, one in stages of 16 channels 2 to 4.
// 64 output channels x 512 pixels in stages of 16 channels (a patch of 32 leaves LDS for one workgroup only):
// 64 -> 64 at 56 x 56, batch 128, data gradient 47 -> 40 us against 256 pixels in stages of 32.
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
constexpr int TAPS = 9;

constexpr int kEpRow = 64 * 2 + 16;     // LDS bytes of an epilogue row: 64 pixels of one channel
constexpr int kEpWave = 32 * kEpRow;    // 32 channels per pass

// ITEMS, GW: see PatchStage; D: steps of filter fragments in flight; EPI: pixels per store; TAIL: the launch may have workgroups that add
// a weight gradient's slices (a form of its own: 64 -> 64 at 56 x 56, batch 128, a step 0.4-1 % less without the branch).
template <int NI, int WM, int WN, int KC, int ITEMS, int GW, int D, int EPI, bool TAIL>
__global__ void __launch_bounds__(256, 2) conv_tile_kernel(GatherParams p)
{
    constexpr int MI = 2;
    constexpr int PT = WN * NI * 32;
    // A stage of KC = 32 channels is 18 steps and comes in two halves of 4 channels per item; one of 16 is 9 steps in one.
    constexpr int KSTEPS = KC / 16, STEPS = TAPS * KSTEPS, KCS = KC + 8, PARTS = KSTEPS;
    static_assert(WM * WN == 4 && STEPS % D == 0 && (KC == 16 || KC == 32), "");
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint32_t buf_bytes = p.buf_bytes;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    // (an image's tiles are as far apart in dispatch order as can be: its last one often has less to do, and
    // neighbouring workgroups go to different XCDs in turn)
    unsigned bx = blockIdx.x, by = blockIdx.y, bz = 0;
    if constexpr (TAIL) {
        if (!conv_block(p, smem, bx, by, bz)) return;
    }
    const int tau = bx / p.ngrp, n_base = (bx - tau * p.ngrp) * p.IPT;
    const int nkb = p.nkb;
    const int ppi = p.Hc * p.Wc;
    const int pix0 = p.IPT > 1 ? 0 : tau * PT;
    const int i0 = fdiv(pix0, p.m_wc);
    const int hin0 = i0 * p.is + p.dhmin;
    const int m0 = (by * WM + wm) * 64;

    PatchStage<ITEMS, GW, KC, 8 / PARTS> in;
    in.init(p, lds0, lds0 + 2 * buf_bytes, n_base, hin0);

    // ---- this lane's pixels
    uint32_t pbase[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int idx = (wn * NI + ni) * 32 + l32;
        int g = 0, px = pix0 + idx;
        bool ok = px < ppi;
        if (p.IPT > 1) {
            g = fdiv(idx, p.m_ppi);
            px = idx - g * ppi;
            ok = g < p.IPT;
        }
        const int i = fdiv(px, p.m_wc), j = px - i * p.Wc;
        pbase[ni] = lds0 + 16u * half + (ok ? (uint32_t)(((g * p.PH + (i - i0) * p.is) * p.PWd + j * p.is) * KCS * 2) : 0u);
    }

    const rsrc_t rs_w = make_rsrc(p.wt, (uint32_t)TAPS * p.Mp * p.KCp * 2u);
    const uint32_t mblks = p.Mp / 32, kstep = mblks * kFrag;
    const uint32_t wlane = m0 < p.Mp ? (uint32_t)(m0 >> 5) * kFrag + lane * 16u : kNoLoad;
    const uint32_t plane_out = (uint32_t)p.Hout * p.Wout;
    const rsrc_t rs_out = make_rsrc(p.out, (uint32_t)p.N * p.M * plane_out * 2u);

    // pixel blocks of this wave that hold any pixel (the last tile of an image: the others are skipped)
    const int nlive = p.IPT > 1 ? NI : max(0, min(NI, (ppi - pix0 - wn * NI * 32 + 31) / 32));

    // All of the workgroup's stages for a wave with NL such blocks (waves of a workgroup may differ: all
    // of them stage, and meet at the same barriers).
    auto run_wave = [&](auto nltag) {
    constexpr int NL = decltype(nltag)::value;
    constexpr int NA = NL > 0 ? NL : 1;
    f32x16 acc[MI][NA];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NA; ++ni)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[mi][ni][j] = 0.f;
    u32x4 wr[D][MI];
#pragma unroll
    for (int q = 0; q < D; ++q)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
            wr[q][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, p.wofs[q / KSTEPS] + (q % KSTEPS) * kstep + mi * kFrag, 0);

    in.start(lds0, buf_bytes);

    for (int s = 0; s < nkb; ++s) {
        const uint32_t buf = (s & 1) ? buf_bytes : 0u, nbuf = buf_bytes - buf;
        uint32_t so = (uint32_t)s * KSTEPS * kstep; // this stage's filter fragments (of tap 0)
        opaque_s(so);
        in.fetch(s + 1, 0); // (past the end: nothing is loaded)
        u32x4 bq[2][NL > 0 ? NL : 1];
#pragma unroll
        for (int ni = 0; ni < NL; ++ni) bq[0][ni] = lds16(pbase[ni] + p.toff[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < STEPS; ++q) {
            if (q + 1 < STEPS) {
#pragma unroll
                for (int ni = 0; ni < NL; ++ni) bq[(q + 1) & 1][ni] = lds16(pbase[ni] + p.toff[(q + 1) / KSTEPS] + 32 * ((q + 1) % KSTEPS));
            }
#pragma unroll
            for (int ni = 0; ni < NL; ++ni)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) {
                    union { u32x4 u; bf16x8 v; } af, bf;
                    af.u = wr[q % D][mi];
                    bf.u = bq[q & 1][ni];
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf.v, af.v, acc[mi][ni], 0, 0, 0);
                }
            // refill the ring with the fragments of step q + D (past the last stage: the next tap's, never used)
            if constexpr (NL > 0) {
                const int q2 = q + D < STEPS ? q + D : q + D - STEPS;
                const uint32_t so2 = p.wofs[q2 / KSTEPS] + so + (q2 % KSTEPS + (q + D < STEPS ? 0 : KSTEPS)) * kstep;
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) wr[q % D][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, so2 + mi * kFrag, 0);
            }
            constexpr int W = STEPS / PARTS; // steps of a part: loads at the first, the pixels to LDS at the last four
            const int h = q / W, qq = q % W;
            if (qq == W - 5) in.align_rows();
            if (qq >= W - 4) {
                in.put_px(nbuf, h, 2 * (qq - (W - 4)));
                in.put_px(nbuf, h, 2 * (qq - (W - 4)) + 1);
            }
            if (qq == W - 1 && h + 1 < PARTS) in.fetch(s + 1, h + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        // on to the other buffer
#pragma unroll
        for (int ni = 0; ni < NL; ++ni) {
            pbase[ni] += nbuf - buf;
            opaque(pbase[ni]);
        }
        __syncthreads();
    }
    // ---- epilogue: bias, bfloat16, NCHW.  Two pixel blocks x 32 channels at a time through LDS (the staging buffers
    // are dead), as [channel][pixel] rows, every wave in a part of its own.
    const uint32_t ep = lds0 + wave * kEpWave;
    uint32_t el = lane; // (what the epilogue computes from the lane is not to be kept through the loop)
    opaque(el);
    const uint32_t eh = el >> 5, e32 = el & 31;
    float bias_tr[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int m = m0 + mi * 32 + e32;
        bias_tr[mi] = (p.bias && m < p.M) ? bf16_to_f32(p.bias[m]) : 0.f;
    }
    constexpr int NIB = NI < 2 ? NI : 2;
    auto store = [&](auto vtag) {
        constexpr int V = decltype(vtag)::value; // pixels per store
        constexpr int LPR = NIB * 32 / V, RPI = 64 / LPR; // lanes of a row; rows per pass over the lanes
#pragma unroll
        for (int pass = 0; pass < (NL + NIB - 1) / NIB; ++pass) {
            const int seg = el % LPR, idx = (wn * NI + pass * NIB) * 32 + seg * V;
            int g = 0, px = pix0 + idx;
            if (p.IPT > 1) {
                g = fdiv(idx, p.m_ppi);
                px = idx - g * ppi;
            }
            const int n = n_base + g;
            const bool px_ok = (px < ppi) & (g < p.IPT) & (n < p.N) & ((int)(pass * NIB + seg * V / 32) < NL);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const float bias = bias_tr[mi];
#pragma unroll
                for (int nb = 0; nb < NIB; ++nb) {
                    if (pass * NIB + nb > NL - 1) break;
                    const f32x16 &a = acc[mi][pass * NIB + nb];
#pragma unroll
                    for (int jq = 0; jq < 4; ++jq)
                        *(lds_u32x2_ptr)(uintptr_t)(ep + e32 * kEpRow + (nb * 32 + 8 * jq + 4 * eh) * 2) =
                            u32x2{f32x2_to_bf16x2(a[4 * jq] + bias, a[4 * jq + 1] + bias), f32x2_to_bf16x2(a[4 * jq + 2] + bias, a[4 * jq + 3] + bias)};
                }
                // (the wave reads what it wrote itself: LDS serves a wave's requests in order)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int it = 0; it < 32 / RPI; ++it) {
                    const int row = it * RPI + el / LPR, m = m0 + mi * 32 + row;
                    const uint32_t off = (px_ok & (m < p.M)) ? ((uint32_t)(n * p.M + m) * plane_out + px) * 2u : kNoLoad;
                    const uint32_t src = ep + row * kEpRow + seg * (V * 2);
                    if constexpr (V == 8) __builtin_amdgcn_raw_buffer_store_b128(lds16(src), rs_out, off, 0, 0);
                    else if constexpr (V == 4) __builtin_amdgcn_raw_buffer_store_b64(*(lds_u32x2_ptr)(uintptr_t)src, rs_out, off, 0, 0);
                    else if constexpr (V == 2) __builtin_amdgcn_raw_buffer_store_b32(*(lds_u32_ptr)(uintptr_t)src, rs_out, off, 0, 0);
                    else __builtin_amdgcn_raw_buffer_store_b16(*(lds_u16_ptr)(uintptr_t)src, rs_out, off, 0, 0);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
    };
    store(std::integral_constant<int, EPI>{});
    };
    if (nlive == NI) run_wave(std::integral_constant<int, NI>{});
    else if (NI > 3 && nlive == NI - 1) run_wave(std::integral_constant<int, (NI > 3 ? NI - 1 : NI)>{});
    else if (2 * nlive > NI) run_wave(std::integral_constant<int, NI>{});
    else if (nlive > 0) run_wave(std::integral_constant<int, (NI + 1) / 2>{});
    else run_wave(std::integral_constant<int, 0>{});
}

template <int NI, int WM, int WN, int KC, int ITEMS, int GW, int D, int EPI, bool TAIL> hipError_t launch_kernel(const GatherParams &p, hipStream_t st)
{
    auto kern = conv_tile_kernel<NI, WM, WN, KC, ITEMS, GW, D, EPI, TAIL>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    dim3 grid(p.tiles_per_img * p.ngrp, (p.Mp / 64 + WM - 1) / WM);
    GatherParams q = p;
    grid = share_grid(q, grid, 256);
    hipLaunchKernelGGL(kern, grid, dim3(256), p.lds_bytes, st, q);
    return hipGetLastError();
}
template <int NI, int WM, int WN, int KC, int ITEMS, int GW, int D, int EPI> hipError_t launch_fixed(const GatherParams &p, hipStream_t st)
{
    return p.tail.blocks ? launch_kernel<NI, WM, WN, KC, ITEMS, GW, D, EPI, true>(p, st) : launch_kernel<NI, WM, WN, KC, ITEMS, GW, D, EPI, false>(p, st);
}
template <int NI, int WM, int WN, int KC, int D, int EPI> hipError_t launch_items(const GatherParams &p, hipStream_t st)
{
    const bool one = p.IPT * p.PH * p.GX * (KC / 8) <= 256;
    if (p.gw == 8) {
        if constexpr (KC == 16) return launch_fixed<NI, WM, WN, KC, 1, 8, D, EPI>(p, st); // (never planned with two items)
        else return one ? launch_fixed<NI, WM, WN, KC, 1, 8, D, EPI>(p, st) : launch_fixed<NI, WM, WN, KC, 2, 8, D, EPI>(p, st);
    }
    if constexpr (KC == 16) return launch_fixed<NI, WM, WN, KC, 1, 7, D, EPI>(p, st);
    else return one ? launch_fixed<NI, WM, WN, KC, 1, 7, D, EPI>(p, st) : launch_fixed<NI, WM, WN, KC, 2, 7, D, EPI>(p, st);
}
template <int NI, int WM, int WN, int KC, int D> hipError_t launch_shape(const GatherParams &p, hipStream_t st)
{
    return p.store_px == 8 ? launch_items<NI, WM, WN, KC, D, 8>(p, st) : p.store_px == 4 ? launch_items<NI, WM, WN, KC, D, 4>(p, st)
           : p.store_px == 2 ? launch_items<NI, WM, WN, KC, D, 2>(p, st) : launch_items<NI, WM, WN, KC, D, 1>(p, st);
}

struct Shape { int ni, wm, wn, kc; hipError_t (*launch)(const GatherParams &, hipStream_t); };
const Shape kShapes[] = {
    {4, 2, 2, 32, launch_shape<4, 2, 2, 32, 3>},
    {4, 4, 1, 32, launch_shape<4, 4, 1, 32, 3>},
    {2, 1, 4, 32, launch_shape<2, 1, 4, 32, 6>},
    {2, 2, 2, 32, launch_shape<2, 2, 2, 32, 6>},
    {2, 4, 1, 32, launch_shape<2, 4, 1, 32, 6>},
    {4, 1, 4, 16, launch_shape<4, 1, 4, 16, 3>}, // 64 channels x 512 pixels: the patch of 32 channels would leave room for one workgroup
};

} // namespace

// Fills the tiling of a nine-tap launch; false when no shape takes it.  *cost_out: clock cycles, roughly.
bool shape_tile(GatherParams &p, int *variant, double *cost_out)
{
    if (p.ntaps != TAPS || p.os != 1) return false;
    GatherParams b = p;
    b.dhmin = b.dwmin = 1 << 30;
    int dhmax = -(1 << 30), dwmax = -(1 << 30);
    for (int t = 0; t < TAPS; ++t) {
        if (p.wtap[t] != t) return false; // (the ring reads a little past a stage's fragments of the first taps)
        b.dhmin = min(b.dhmin, p.dh[t]); dhmax = max(dhmax, p.dh[t]);
        b.dwmin = min(b.dwmin, p.dw[t]); dwmax = max(dwmax, p.dw[t]);
    }
    b.PWd = (p.Wc - 1) * p.is + (dwmax - b.dwmin) + 1;
    b.ksplit = 1; b.T = 1; b.part = nullptr;
    const int ppi = p.Hc * p.Wc;
    if (!divides_exactly(ppi, p.Wc)) return false; // (a pixel's row and column)
    b.m_wc = magic_of(p.Wc); b.m_ppi = magic_of(ppi); b.m_pwd = magic_of(b.PWd);
    b.gw = p.Win % 2 ? 7 : 8;
    b.GX = (p.Win + b.gw - 1) / b.gw;
    b.m_gx = magic_of(b.GX);
    b.store_px = ppi % 8 == 0 ? 8 : ppi % 4 == 0 ? 4 : ppi % 2 == 0 ? 2 : 1;
    int f = -1, f_ipt = 0;
#ifdef CAC_TUNING
    if (const char *force = getenv("CAC_TILE_SHAPE")) sscanf(force, "%d,%d", &f, &f_ipt);
#endif
    GatherParams best{};
    double best_cost = 1e300;
    for (int v = 0; v < (int)(sizeof(kShapes) / sizeof(kShapes[0])); ++v) {
        if (f >= 0 && v != f) continue;
        const Shape &sh = kShapes[v];
        if (sh.wm * 64 > b.Mp && sh.wm > 1) continue;
        GatherParams q = b;
        const int pt = sh.wn * sh.ni * 32, kcs = sh.kc + 8; // (LDS elements per patch pixel: an odd number of 16-byte units)
        q.KCp = (p.KCin + sh.kc - 1) / sh.kc * sh.kc;
        q.nkb = q.kbs = q.KCp / sh.kc;
        q.IPT = 2 * ppi <= pt ? pt / ppi : 1;
        if (f_ipt) q.IPT = f_ipt;
        if (q.IPT > 1) {
            q.tiles_per_img = 1;
            q.PH = (q.Hc - 1) * q.is + (dhmax - q.dhmin) + 1;
        } else {
            q.tiles_per_img = (ppi + pt - 1) / pt;
            const int rows = min(q.Hc, (pt + q.Wc - 2) / q.Wc + 1);
            q.PH = (rows - 1) * q.is + (dhmax - q.dhmin) + 1;
        }
        const int items = q.IPT * q.PH * q.GX * (sh.kc / 8);
        if (items > (sh.kc == 16 ? 256 : 512)) continue;
        q.patch_px = q.IPT * q.PH * q.PWd;
        q.buf_bytes = max(q.patch_px * kcs * 2, 2 * kEpWave);
        q.lds_bytes = 2 * q.buf_bytes + kDumpBytes;
        if (q.lds_bytes > 160 * 1024) continue;
        q.m_ph = magic_of(q.PH);
        for (int t = 0; t < TAPS; ++t) {
            q.wofs[t] = (uint32_t)t * (q.KCp / 16) * (q.Mp / 32) * kFrag;
            q.toff[t] = (uint32_t)((p.dh[t] - q.dhmin) * q.PWd + (p.dw[t] - q.dwmin)) * kcs * 2u;
        }
        q.ngrp = (q.N + q.IPT - 1) / q.IPT;
        const int mtiles = (q.Mp / 64 + sh.wm - 1) / sh.wm;
        const long wgs = (long)q.tiles_per_img * q.ngrp * mtiles;
        q.gpw = 1;
        // Few workgroups: conv_wave.hip, whose waves share out the channels of a tile, and the launches of conv_mfma.hip are the
        // faster ones (against the latter: 512 -> 512 at 4 x 4, batch 128, 64 workgroups here: 28 against 38 us;
        // 240 -> 272 at 12 x 12, batch 24, 144 workgroups: 2 us; 128 -> 128 at 16 x 16, batch 128, 256 workgroups: even).
        // For rows of odd length they need an element-by-element repack, for planes that are no multiple of 4 pixels
        // they store single elements, and lose from 64 workgroups on (512 -> 512 at 7 x 7, batch 64, 104 workgroups:
        // 43.2 against 41.5 us; 72 -> 100 at 27 x 30, batch 24, 192 workgroups: 25 against 18 us).
        if (f < 0 && wgs < (p.Win % 2 || ppi % 4 ? 64 : 160)) continue;
        // Cycles of a compute unit.  A stage is 18 steps of 2 x NI MFMAs of 32 cycles, of which a pair of resident
        // workgroups keeps the matrix pipe busy for the fractions measured (a single one for less); a wave's last
        // tile may have fewer live blocks; each pair pays a start and an epilogue.
        double live = 0;
        for (int t = 0; t < q.tiles_per_img; ++t) live += min(sh.ni, ((q.IPT > 1 ? pt : ppi - t * pt) + 31) / 32);
        live /= (double)q.tiles_per_img * sh.ni;
        const double k = (double)((wgs + 255) / 256);
        const bool pairs = k > 1 && q.lds_bytes <= 80 * 1024;
        // (stages of 16 channels: twice the barriers; in rows of odd length the shifts of a whole item come at once)
        const double eff = sh.ni == 4 ? (pairs ? (sh.kc == 16 ? 0.70 : 0.78) : 0.55) / (sh.kc == 16 && q.gw == 7 ? 1.35 : 1.0)
                                      : (pairs ? (sh.wm == 4 ? 0.50 : 0.52) : 0.45);
        const double twice = items > 256 ? 1.1 : 1.0;
        const double cost = k * q.nkb * (TAPS * (sh.kc / 16)) * 2.0 * sh.ni * 32 * live * twice / eff + (pairs ? (k + 1) / 2 : k) * 6000.0;
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

hipError_t launch_tile(const GatherParams &p, int variant, hipStream_t st) { return kShapes[variant].launch(p, st); }

int describe_tile(const GatherParams &p, int variant, char *buf, size_t len)
{
    const Shape &v = kShapes[variant];
    const int mt = (p.Mp / 64 + v.wm - 1) / v.wm;
    return snprintf(buf, len, "tile=%dch x %dpx (NI=%d WM=%d WN=%d) taps=%d img/tile=%d patch=%dx%d units/wg=%d grid=%dx%dx1 lds=%dB, input read in place",
                    64 * v.wm, 32 * v.ni * v.wn, v.ni, v.wm, v.wn, p.ntaps, p.IPT, p.PH, p.PWd, 1, p.tiles_per_img * p.ngrp, mt, p.lds_bytes);
}

} // namespace cac
