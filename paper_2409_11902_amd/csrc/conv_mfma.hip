// Forward convolution and data gradient (forward / data-gradient formulas of the
// compression figure; neither depends on the compressed activation) as one MFMA
// implicit GEMM.
//
// Both are the same "gather" sum
//   out[n, m, h, w] = bias[m] + sum_t sum_kc Wt[t][m][kc] * in[n, i*is + dh_t, j*is + dw_t, kc]
// over a list of taps t, for the output pixels (h, w) = (i*os + a0, j*os + b0):
//   forward:            in = X,  m = o, kc = c, os = 1, is = stride, (dh, dw) = (r - pad, s - pad)
//   data gradient, s=1: in = dY, m = c, kc = o, os = 1, is = 1,      (dh, dw) = (pad - r, pad - s)
//   data gradient, s=2: one launch per output parity class (a0, b0) with the
//                       taps whose (a0 + pad - r) and (b0 + pad - s) are even.
// The reduction index kc must be contiguous per pixel for the MFMA operand
// layout.  In LDS it always is; on the way there the input takes one of two
// routes: a channels-last copy in the workspace (repack_kernel) that the GEMM's
// copy waves move in 16-byte pieces, or -- where that copy would be the larger
// part of the repack launch -- no copy at all: the copy waves read 8 channel x
// 8 pixel blocks of the tensor as it lies and transpose them in registers.  The
// filter is always repacked into MFMA fragment order, padded with zeros to
// multiples of 16 channels (same launch; the forward pass forms the 2 x 2 pooled
// map there too where the tiles are whole).  The GEMM is conv_gather_kernel (conv_gather.h).
#include <stdio.h>
#include <stdlib.h>

#include "common.h"
#include "conv_mfma.h"
#include "dw_reduce.h"
#include "filter_repack.h"

namespace cac {

namespace {

using gather::KC;
using gather::KCS;
using gather::kMaxItems;

// ---- repacks ---------------------------------------------------------------------

__global__ void __launch_bounds__(256) repack_kernel(RepackParams p)
{
    __shared__ bf16_t sm[kRepackElems];
    repack_body(p, blockIdx.x, sm, threadIdx.x);
}

// The input and filter repacks of one call.
// N 0: the filter alone.  Z, Wimg: see RepackParams (Z null: no pooling; else HW must be a multiple of 2*Wimg and Wimg 4 or a multiple of 8).
RepackParams make_repack(const bf16_t *in, bf16_t *out, int N, int C, int HW, int Cp, const bf16_t *W, bf16_t *Wt, int O,
                         int Cw, int RS, int Mp, int KCp, int transpose, bf16_t *Z, int Wimg, int decim = 0)
{
    RepackParams p{};
    p.in = in; p.out = out; p.N = N; p.C = C; p.HW = HW; p.Cp = Cp;
    p.Z = Z; p.Wimg = Wimg; p.decim = decim;
    p.fast = HW % 2 == 0; // planes start at multiples of 4 bytes: 16-byte loads need no more
    const int cgs = Cp / 8, cgw = cgs < 8 ? cgs : 8;
    const long items = p.fast ? (long)N * ((cgs + cgw - 1) / cgw) * cgw * (Z && Wimg != 4 ? HW / 16 : (HW + 7) / 8) : 0;
    // (a thread's loads are all in flight at once, so a small input is bound by latency, not by
    // the number of waves per compute unit: give every unit a wave before any gets a second)
    p.in_wpb = items > 64 * 256 ? 4 : 1; // (measured: two waves per block are slower than either)
    p.in_blocks = p.fast ? (int)((items + 64 * p.in_wpb - 1) / (64 * p.in_wpb)) : N * ((Cp + 63) / 64) * ((HW + 63) / 64);
    p.f = FilterRepack{W, Wt, O, Cw, RS, Mp, KCp, transpose};
    return p;
}
// The repacks of a data-gradient call and, in the blocks after them, the slice sum that the weight gradient of the same layer has
// left over: two small, independent pieces of a backward pass that would otherwise each pay for a launch.
template <int SY, int V> __global__ void __launch_bounds__(256) repack_reduce_kernel(RepackParams p, unsigned nrep, DwReduceTail t)
{
    __shared__ __align__(16) bf16_t sm[kRepackElems];
    if (blockIdx.x < nrep) repack_body(p, blockIdx.x, sm, threadIdx.x);
    else dw_reduce_body<SY, V, 1>(t, blockIdx.x - nrep, 0, threadIdx.x, sm);
}

// tail: a deferred weight-gradient slice sum to run in the same launch, or null.
hipError_t launch_repack(const RepackParams &p, hipStream_t st, const DwReduceTail *tail = nullptr)
{
    if (tail && tail->blocks) {
        const DwReduceTail &t = *tail;
        const unsigned nrep = p.blocks();
#define CAC_RR(SY, V) hipLaunchKernelGGL((repack_reduce_kernel<SY, V>), dim3(nrep + t.blocks), dim3(256), 0, st, p, nrep, t)
        if (t.V == 4) {
            if (t.SY == 16) CAC_RR(16, 4);
            else if (t.SY == 4) CAC_RR(4, 4);
            else CAC_RR(1, 4);
        } else {
            if (t.SY == 16) CAC_RR(16, 1);
            else if (t.SY == 4) CAC_RR(4, 1);
            else CAC_RR(1, 1);
        }
#undef CAC_RR
        return hipGetLastError();
    }
    hipLaunchKernelGGL(repack_kernel, dim3(p.blocks()), dim3(256), 0, st, p);
    return hipGetLastError();
}

int round_up(int x, int m) { return (x + m - 1) / m * m; }

// Chooses the workgroup shape and fills the tiling; false if no shape fits.
//
// Candidates: waves along m (wm) x pixel blocks per wave (ni), and, where the output is written
// in whole planes, the number of workgroups that share a tile's channel blocks (their float sums
// go to the workspace and gather_finish_kernel adds them up).  Each is priced with a rough model
// in clock cycles: a step (one tap, 16 channels) costs a wave 32 cycles per MFMA but at least the
// time the CU's vector cache needs for the four waves' filter fragments; a workgroup pays a fixed
// start-up and epilogue; the chip runs 256 workgroups at a time; all filter and input bytes have
// to come through L2; shared-out channels cost a second kernel and the traffic of the sums.
bool shape_gather(GatherParams &p, int *variant)
{
    p.dhmin = p.dwmin = 1 << 30;
    int dhmax = -(1 << 30), dwmax = -(1 << 30);
    for (int t = 0; t < p.ntaps; ++t) {
        p.dhmin = min(p.dhmin, p.dh[t]); dhmax = max(dhmax, p.dh[t]);
        p.dwmin = min(p.dwmin, p.dw[t]); dwmax = max(dwmax, p.dw[t]);
    }
    p.PWd = (p.Wc - 1) * p.is + (dwmax - p.dwmin) + 1;
    p.nkb = (p.KCp + KC - 1) / KC;
    p.part = nullptr;
    const int ppi = p.Hc * p.Wc;
    if (!divides_exactly(ppi, p.Wc)) return false; // (a pixel's row and column)
    p.m_wc = magic_of(p.Wc); p.m_ppi = magic_of(ppi); p.m_pwd = magic_of(p.PWd);
    const bool whole_planes = p.os == 1 && p.Hc == p.Hout && p.Wc == p.Wout && ppi % 4 == 0;
    const char *force = nullptr;
    int f_wm = 0, f_ni = 0, f_ks = 0;
#ifdef CAC_TUNING // development builds: CAC_GATHER_SHAPE="wm,ni,ksplit" overrides the model
    force = getenv("CAC_GATHER_SHAPE");
    if (force) sscanf(force, "%d,%d,%d", &f_wm, &f_ni, &f_ks);
#endif
    GatherParams best{};
    double best_cost = 1e300;
    int best_variant = 0;
    for (int wm : {4, 2, 1}) {
        if (wm * 64 > p.Mp && wm > 1) continue;
        const int wn = 4 / wm;
        for (int ni : {2, 1}) { // (NI = 4 fits the register file only with spills and measured slower)
            GatherParams q = p;
            const int pt = wn * ni * 32;
            q.IPT = 2 * ppi <= pt ? pt / ppi : 1;
            if (q.IPT > 1) {
                q.tiles_per_img = 1;
                q.PH = (q.Hc - 1) * q.is + (dhmax - q.dhmin) + 1;
            } else {
                q.tiles_per_img = (ppi + pt - 1) / pt;
                const int rows = min(q.Hc, (pt + q.Wc - 2) / q.Wc + 1); // class-grid rows a tile can touch
                q.PH = (rows - 1) * q.is + (dhmax - q.dhmin) + 1;
            }
            q.patch_px = q.IPT * q.PH * q.PWd;
            if (q.patch_px * (KC / 8) > 256 * kMaxItems) continue;
            if ((long)2 * q.patch_px * KCS * 2 > 110 * 1024) continue; // (leaves room for the epilogue's transpose)
            // Few taps: several 32-channel groups per pass, which the kernel treats as further taps,
            // so that taps x groups is 4 or 8 and the kernels with the deep operand rings apply
            // (with one or two taps a pass is otherwise a handful of MFMAs, and the filter
            // fragments, requested two steps ahead, arrive long after they are wanted).  As many
            // groups as the channels, LDS and the copy threads' registers allow -- and, where the
            // input could be read in place with one group, only as many as still allow that.
            q.T = 1;
            const int items_in_place = q.IPT * q.PH * ((q.Win + 7) / 8) * (KC / 8);
            for (int t : {4, 2}) {
                if ((q.ntaps * t != 8 && q.ntaps * t != 4) || KC * (t - 1) >= q.KCp) continue;
                if (q.patch_px * (KC / 8) * t > 256 * kMaxItems) continue;
                if ((long)2 * q.patch_px * (KC * t + 8) * 2 > 124 * 1024) continue; // (with the wide stores' 36 KB still inside the CU's 160 KB)
                if (items_in_place <= 512 && items_in_place * t > 512) continue;
                q.T = t;
                break;
            }
            q.t_log2 = q.T == 4 ? 2 : q.T == 2 ? 1 : 0;
            q.kcs = KC * q.T + 8;
            q.nkb = (q.KCp + KC * q.T - 1) / (KC * q.T);
            q.m_img = magic_of(q.PH * q.PWd);
            q.m_gx = magic_of((q.Win + 7) / 8); q.m_ph = magic_of(q.PH);
            q.ngrp = (q.N + q.IPT - 1) / q.IPT;
            const int mtiles = (q.Mp / 64 + wm - 1) / wm;
            const long wgs1 = (long)q.tiles_per_img * q.ngrp * mtiles;
            for (int ks = 1; ks <= (whole_planes ? q.nkb : 1); ++ks) {
                if (q.nkb % ks) continue;
                if (force && (wm != f_wm || ni != f_ni || ks != f_ks)) continue;
                q.ksplit = ks;
                q.wide_store = whole_planes && ks == 1 && ppi % 8 == 0; // 16-byte runs of pixels, aligned
                q.kbs = q.nkb / ks;
                q.m_kbs = magic_of(q.kbs);
                // a few units per workgroup (a longer pipeline) as long as every CU still gets a workgroup
                q.gpw = (int)max(1L, min((long)((8 + q.kbs - 1) / q.kbs), wgs1 * ks / 256));
                if (!divides_exactly((uint64_t)q.gpw * q.kbs, q.kbs)) continue; // (a stage's unit: beyond 2^16 channel blocks)
                const long runs = (q.ngrp + q.gpw - 1) / q.gpw;
                const long wgs = (long)q.tiles_per_img * runs * mtiles * ks;
                // cycles per step as measured (vector-cache bound below NI = 4), two-step prefetch 1.35 x
                // (without the deep rings a step waits for its filter fragments: measured 700-1000 cycles;
                // with them on few taps, where every fragment is used once, 500-600)
                const int ntt = q.ntaps * q.T;
                const double step = ntt == 9 ? (ni == 1 ? 150.0 : 235.0) : (ntt == 4 || ntt == 8) ? (ni == 1 ? 500.0 : 600.0) : 800.0;
                const double t_wg = (double)q.gpw * q.kbs * 2 * q.ntaps * q.T * step + 8000.0;
                const double l2_bytes = (double)wgs * q.gpw * q.kbs * KC * q.T * 2.0 * (q.ntaps * 64.0 * wm + q.patch_px);
                double cost = max((double)((wgs + 255) / 256) * t_wg, l2_bytes / 6000.0 + 8000.0);
                cost += l2_bytes / 6000.0 * 0.01; // between equals, the one that moves less
                if (ks > 1) cost += 6000.0 + (double)ks * q.N * q.M * ppi * 8.0 / 2500.0;
                if (cost < best_cost) {
                    best_cost = cost;
                    best = q;
                    best_variant = (ni == 2 ? 0 : 3) + (wm == 1 ? 0 : wm == 2 ? 1 : 2);
                }
            }
        }
    }
    if (best_cost > 1e299) return false;
    p = best;
    *variant = best_variant;
    return true;
}

hipError_t run_gather(const GatherParams &p, int variant, hipStream_t st)
{
    switch (p.tile) {
    case 1: return launch_tile(p, variant, st);
    case 2: return launch_dx2(p, variant, st);
    case 3: return launch_pw(p, variant, st);
    case 4: return launch_wave(p, variant, st);
    case 5: return launch_wave_dx2(p, variant, st);
    }
    return p.tail.blocks ? launch_conv_gather_tail(p, variant, st) : launch_conv_gather(p, variant, st);
}

bool supported(const Geom &g, int dtype)
{
    if (dtype != CAC_BF16) return false;
    if (g.R * g.S > 9) return false;
    if (g.sh != g.sw || (g.sh != 1 && g.sh != 2)) return false;
    // 32-bit byte offsets with 2^31 reserved for "no load"
    const long lim = 1L << 30;
    if ((long)g.N * g.H * g.W * round_up(g.C, 16) >= lim || (long)g.N * g.P * g.Q * round_up(g.K, 16) >= lim) return false;
    if ((long)g.R * g.S * round_up(g.K, 64) * round_up(g.C, 64) >= lim) return false;
    return true;
}

bool use_tile()
{
#ifdef CAC_TUNING
    if (const char *f = getenv("CAC_TILE")) return atoi(f) != 0;
#endif
    return true;
}

// A 1 x 1 stride-1 launch: conv_pw.hip (p.tile = 3), or the gather where that is the faster one and can (rows that fit LDS).
bool plan_pw(GatherParams &p, bool pool, bool record_free, int *variant)
{
    GatherParams pw = p, ga = p;
    int pw_variant, ga_variant;
    bool gather, gather_whole;
    if (!shape_pw(pw, pool, record_free, &pw_variant, &gather, &gather_whole)) return false;
    gather = (gather || gather_whole) && shape_gather(ga, &ga_variant) && (gather || ga.ksplit == 1);
    p = gather ? ga : pw;
    p.tile = gather ? 0 : 3;
    *variant = gather ? ga_variant : pw_variant;
    return true;
}

// A launch with other filters: nine taps go to conv_tile.hip, or with few pixels to conv_wave.hip, what they leave to the gather.
bool plan_other(const Geom &g, GatherParams &p, bool fwd, int *variant)
{
    GatherParams wave = p, tile = p;
    int wave_variant;
    double wave_cost, tile_cost = 1e300;
    const bool have_tile = use_tile() && shape_tile(tile, variant, &tile_cost); // (*variant: its own until another is chosen)
    bool have_wave = use_tile() && shape_wave(wave, &wave_variant, &wave_cost);
    // Where conv_tile.hip has no shape, 300 random layers took 0.59 of the gather's time with waves (both directions, 9 of them over
    // 1.05).  Two lines remain to the gather: sums over 48 channels and less, which leave a wave without a stage (data
    // gradients 1.0-1.09 of the time; forward passes up to 4096 pixels 0.7, the input's copy falls away), and a dozen tiles of
    // less than 0.1 GFLOP, launches and start-up either way, where it shares the channels over workgroups.
    const long px = (long)p.N * p.Hc * p.Wc;
    const bool few = (p.KCin <= 48 && (!fwd || px >= 4096)) || (p.KCin <= 256 && (px + 63) / 64 * (p.Mp / 64) <= 12 && 18.0 * px * p.KCin * p.M < 1e8);
    // Long sums over few workgroups where a lane stages two items of eight channels, under stride 2 (twice the rows) and on rows past 40
    // pixels or so: stage after stage of a wave, where the gather shares the channels out.  Under stride 2 the waves took 1.0 to 1.5 of
    // its time from twelve stages a wave on (1600 -> 41 at 12 x 12, batch 22: 39 against 25 us).  Of 196 random layers with
    // fewer, the 40 with six and more, at most 32 workgroups and an input whose copy the gather makes in whole items took 1.1 (592 -> 27
    // at 5 x 48, batch 2: 23.6 against 17.0; four below 0.95), the others 0.81 (10 over 1.05).  Under stride 1 the three such layers of
    // 1000 took 1.03, 1.10 and 1.45 (data gradient of 32 -> 1344 at 16 x 47, batch 2: 30.1 against 20.8).
    const bool two = have_wave && wave.IR * wave.GX * (wave.KCp / wave.nkb) > 64 * 8;
    const bool long_sums = (p.is == 2 && wave.kbs >= 12) ||
                           ((p.is == 2 || two) && wave.kbs >= 6 && wave.tiles_per_img * wave.mtiles <= 32 && p.Hin * p.Win % 2 == 0);
    if (GatherParams gather = p; have_wave && long_sums && !have_tile && shape_gather(gather, variant) && gather.ksplit > 1) {
        p = gather;
        return true;
    }
    if (GatherParams gather = p; have_wave && few && (have_tile || shape_gather(gather, variant))) {
        have_wave = false;
        if (!have_tile) {
            p = gather;
            return true;
        }
    }
    // What only the waves take with matrix instructions (few pixels or few channels) is theirs where conv_lds.hip or the plain kernel are not
    // faster: few terms, or more padding than channels.  A forward pass has the filter laid out in the launch that pools, a data gradient by
    // a launch of its own, 5 us, or for nothing in that of the weight gradient.  363 random layers, by waves against without: data gradients 1.01
    // of the time, half of them over 1.05 (3 -> 3 at 1 x 1, batch 6, 10.7 against 3.9 us), forward passes 0.54, a third over 1.05 (1 -> 6 at
    // 56 x 56, stride 2, batch 221, 69 against 11); with this line 0.73 (3 of 87 over 1.05, the worst 1.17) and 0.48 (none).  Both gradients
    // in a call 0.73 by waves, 18 of 87 over 1.05; 0.71 and none.
    if (GatherParams gather = p; have_wave && !have_tile && cost_without_mfma(g, CAC_BF16, !fwd) < 0.85e-3 * wave_cost + (fwd ? 0.0 : 5.0) &&
                                 !shape_gather(gather, variant))
        return false;
    // Against conv_tile.hip by the ratio of the two planners' cycles, which counts a stage alike for one item to a lane and for two.
    // One: 200 random layers, below 0.55 the waves take 0.76 of the time (48 layers, 2 of them over 1.05), up to 0.7 it is 1.0, above 1.0
    // 1.6.  Two: under stride 1 0.8 below 0.45 and 1.04 from there to 0.55 (19 layers; data gradient of 67 -> 464 at 51 x 51, batch 7:
    // 44.7 against 39.1 us), under stride 2 0.8 below 0.50 and 1.0 from there to 0.55 (57 layers).
    if (have_wave && have_tile) have_wave = wave_cost < (!two ? 0.55 : p.is == 1 ? 0.45 : 0.50) * tile_cost;
#ifdef CAC_TUNING
    if (const char *f = getenv("CAC_WAVE"); f && atoi(f) == 0) have_wave = false;
#endif
    if (have_wave) {
        p = wave;
        p.tile = 4;
        *variant = wave_variant;
        return true;
    }
    if (have_tile) {
        p = tile;
        p.tile = 1;
        return true;
    }
    return shape_gather(p, variant);
}

// Whole 2 x 2 tiles, rows a multiple of 8 pixels: the pooled map falls out of the repack.
bool record_in_repack(const Geom &g) { return !g.pmax && g.kh == 2 && g.kw == 2 && g.H % 2 == 0 && (g.W % 8 == 0 || g.W == 4); }

// Forward pass as a gather GEMM: output channels x output pixels, taps (r - ph, s - pw).
bool plan_fwd(const Geom &g, int dtype, GatherParams &p, int *variant)
{
    if (!supported(g, dtype)) return false;
    p = GatherParams{};
    p.N = g.N; p.M = g.K; p.Mp = round_up(g.K, 64); p.KCp = round_up(g.C, 16);
    p.Hin = g.H; p.Win = g.W; p.Hout = g.P; p.Wout = g.Q; p.Hc = g.P; p.Wc = g.Q;
    p.os = 1; p.a0 = p.b0 = 0; p.is = g.sh;
    p.ntaps = p.ntaps_total = g.R * g.S;
    for (int r = 0; r < g.R; ++r)
        for (int s = 0; s < g.S; ++s) {
            const int t = r * g.S + s;
            p.dh[t] = r - g.ph; p.dw[t] = s - g.pw; p.wtap[t] = t;
        }
    // A 1 x 1 filter with stride 2 reaches one pixel of every 2 x 2 tile.  Where the repack launch goes
    // over those tiles anyway (it forms the 2 x 2 pooled map: rows a multiple of 8 pixels, an even
    // number of them), its channels-last copy keeps just that pixel: a quarter of the bytes to write
    // and to stage, and the GEMM sees a stride-1 layer on an image of half the extent.
    p.decim = g.R == 1 && g.S == 1 && g.sh == 2 && g.sw == 2 && g.ph == 0 && g.pw == 0 && g.kh == 2 && g.kw == 2 &&
              !g.pmax && g.H % 2 == 0 && g.W % 8 == 0;
    if (p.decim) {
        p.Hin = g.H / 2; p.Win = g.W / 2; p.is = 1;
    }
    p.KCin = g.C;
    if (use_tile() && plan_pw(p, !g.pmax && g.kh == 2 && g.kw == 2, record_in_repack(g), variant)) {
        if (!p.tile) return true;
        p.w_direct = p.w_direct && g.C % 16 == 0; // (rows of W are whole fragments)
        p.w_kstep = p.w_direct ? 32u : (uint32_t)p.Mp * 32u;
        p.w_bytes = p.w_direct ? (uint32_t)g.K * g.C * 2u : (uint32_t)p.Mp * p.KCp * 2u;
        return true;
    }
    return plan_other(g, p, true, variant);
}

// Data gradient: one gather GEMM (input channels x input pixels) per parity class of the input
// pixel, each with the taps that reach that class.  Every class is planned before anything is
// launched.  *empty_class: some class has no tap at all (stride > filter) and stays zero.
bool plan_dx(const Geom &g, int dtype, GatherParams &base, GatherParams (&cls)[4], int (&variant)[4], int *ncls, bool *empty_class)
{
    if (!supported(g, dtype)) return false;
    base = GatherParams{};
    base.N = g.N; base.M = g.C; base.Mp = round_up(g.C, 64); base.KCp = round_up(g.K, 16);
    base.Hin = g.P; base.Win = g.Q; base.Hout = g.H; base.Wout = g.W;
    base.os = g.sh; base.is = 1; base.ntaps_total = g.R * g.S;
    *ncls = 0;
    *empty_class = false;
    // One launch for the four classes: by waves or with shared stages.  The two estimates, in cycles, cross where the measured
    // times do: over 142 random layers that both take, waves needed 0.37 to 0.82 of the other kernel's time where the ratio of the
    // estimates is below 0.5 (79 layers, the worst 0.98), 0.99 up to 0.6, 1.0 up to 0.7 and up to twice the time above (short sums over
    // many tiles: 1760 -> 32 at 28 x 26 of dY, batch 9, 41 us there, 89 by waves).  Odd rows only waves take.
    GatherParams wave = base, dx2 = base;
    wave.KCin = dx2.KCin = g.K;
    int wave_variant;
    double wave_cost, dx2_cost = 1e300;
    const bool have_dx2 = use_tile() && shape_dx2(g, dx2, &variant[0], &dx2_cost);
    bool have_wave = use_tile() && shape_wave_dx2(g, wave, &wave_variant, &wave_cost);
    if (have_wave && have_dx2) have_wave = wave_cost < 0.5 * dx2_cost;
    if (have_wave || have_dx2) {
        GatherParams &p = cls[(*ncls)++];
        p = have_wave ? wave : dx2;
        p.tile = have_wave ? 5 : 2;
        if (have_wave) variant[0] = wave_variant;
        base.KCp = p.KCp;
        return true;
    }
    for (int a0 = 0; a0 < g.sh; ++a0)
        for (int b0 = 0; b0 < g.sw; ++b0) {
            GatherParams p = base;
            p.a0 = a0; p.b0 = b0;
            p.Hc = (g.H - a0 + g.sh - 1) / g.sh;
            p.Wc = (g.W - b0 + g.sw - 1) / g.sw;
            if (p.Hc <= 0 || p.Wc <= 0) continue;
            p.ntaps = 0;
            for (int r = 0; r < g.R; ++r)
                for (int s = 0; s < g.S; ++s) {
                    const int th = a0 + g.ph - r, tw = b0 + g.pw - s;
                    if (th % g.sh || tw % g.sw) continue; // C++ remainder: zero iff divisible, also for negatives
                    p.dh[p.ntaps] = th / g.sh; p.dw[p.ntaps] = tw / g.sw; p.wtap[p.ntaps] = r * g.S + s;
                    ++p.ntaps;
                }
            if (p.ntaps == 0) { *empty_class = true; continue; }
            p.KCin = g.K;
            if (use_tile() && plan_pw(p, false, false, &variant[*ncls])) {
                p.w_direct = 0;
                p.w_kstep = (uint32_t)p.Mp * 32u;
                p.w_bytes = (uint32_t)p.Mp * p.KCp * 2u;
            } else if (!plan_other(g, p, false, &variant[*ncls])) return false;
            else if (p.tile) base.KCp = p.KCp; // (nine taps of one class are all taps: it is the only one)
            cls[(*ncls)++] = p;
        }
    return true;
}

// The data gradient reads dY where it lies when every class's patch splits into at most 512
// items of 8 x 8 elements (rows of an even number of pixels): no channels-last copy, only the
// filter repack.  It pays where the copy is the larger part of the repack launch (measured:
// 3.8 us gained per call at 230 input elements per filter element, 1.5 us lost at 3.5).
bool dx_reads_in_place(const Geom &g, const GatherParams (&cls)[4], int ncls)
{
    if (ncls == 1 && cls[0].tile) return true;
    bool direct = g.Q % 2 == 0 && (long)g.N * g.K * g.P * g.Q >= 8L * g.R * g.S * g.K * g.C;
    for (int k = 0; k < ncls; ++k) direct = direct && cls[k].IPT * cls[k].PH * ((g.Q + 7) / 8) * (KC / 8) * cls[k].T <= 512;
    return direct;
}

int describe_one(const GatherParams &p, int variant, char *buf, size_t len)
{
    if (p.tile == 3) return describe_pw(p, variant, buf, len);
    if (p.tile == 4) return describe_wave(p, variant, buf, len);
    if (p.tile == 5) return describe_wave_dx2(p, variant, buf, len);
    if (p.tile) return p.tile == 2 ? describe_dx2(p, variant, buf, len) : describe_tile(p, variant, buf, len);
    static const int shape[6][3] = {{2, 1, 4}, {2, 2, 2}, {2, 4, 1}, {1, 1, 4}, {1, 2, 2}, {1, 4, 1}}; // NI, WM, WN
    const int *v = shape[variant];
    const int runs = (p.ngrp + p.gpw - 1) / p.gpw, mt = (p.Mp / 64 + v[1] - 1) / v[1];
    return snprintf(buf, len, "gather tile=%dch x %dpx (NI=%d WM=%d WN=%d) taps=%d ch/pass=%d img/tile=%d patch=%dx%d units/wg=%d grid=%dx%dx%d lds=%dB",
                    64 * v[1], 32 * v[0] * v[2], v[0], v[1], v[2], p.ntaps, KC * p.T, p.IPT, p.PH, p.PWd, p.gpw, p.tiles_per_img * runs, mt,
                    p.ksplit, 2 * p.patch_px * p.kcs * 2 + (p.wide_store ? 4 * 64 * ((v[0] < 2 ? v[0] : 2) * 64 + 16) : 0));
}

// The forward launch reads X where it lies: the kernels made for it, and the gather under the same conditions as dY in the
// data gradient.  (A pooled map that falls out of the repack launch then does so without the channels-last copy.)
bool fwd_reads_in_place(const Geom &g, const GatherParams &p)
{
    return p.tile || (!p.decim && g.W % 2 == 0 && (long)g.N * g.C * g.H * g.W >= 8L * g.R * g.S * g.K * g.C &&
                      p.IPT * p.PH * ((g.W + 7) / 8) * (KC / 8) * p.T <= 512);
}

// The record's own launch carries the filter's repack: nothing else forms the one, and the other is a launch for nothing else.
bool record_with_filter(const Geom &g, const GatherParams &p)
{
    return (p.tile == 3 ? !p.w_direct && !p.pw_pool : fwd_reads_in_place(g, p) && !record_in_repack(g)) && compress_fast_covers(g, CAC_BF16);
}

// Workspace: [channels-last input][repacked filter][float sums of shared-out channels], each
// part starting at a multiple of 256 bytes; nothing for an operand that is read where it lies.
struct WsLayout { size_t in, wt, part; };
WsLayout ws_layout(size_t in_elems, size_t wt_elems, const GatherParams &p)
{
    auto up = [](size_t n) { return (n + 255) / 256 * 256; };
    WsLayout l;
    l.in = up(in_elems * 2);
    l.wt = up(wt_elems * 2);
    l.part = p.ksplit > 1 ? (size_t)p.ksplit * p.N * p.M * p.Hc * p.Wc * sizeof(float) : 0;
    return l;
}
WsLayout fwd_layout(const Geom &g, const GatherParams &p)
{
    const size_t in = (size_t)p.N * p.Hin * p.Win * p.KCp; // (Hin, Win: of the pixels a decimated copy keeps)
    return ws_layout(fwd_reads_in_place(g, p) ? 0 : in, p.w_direct ? 0 : (size_t)p.ntaps_total * p.Mp * p.KCp, p);
}
WsLayout dx_layout(const Geom &g, const GatherParams &base, const GatherParams (&cls)[4], int ncls)
{
    const size_t in = (size_t)base.N * base.Hin * base.Win * base.KCp;
    // (only a stride-1 data gradient, a single class, ever shares out its channels)
    return ws_layout(dx_reads_in_place(g, cls, ncls) ? 0 : in, (size_t)base.ntaps_total * base.Mp * base.KCp, ncls == 1 ? cls[0] : base);
}

} // namespace

bool describe_conv_mfma(const Geom &g, int dtype, bool data_grad, char *buf, size_t len)
{
    GatherParams p{}, cls[4];
    int variant[4], ncls = 0;
    bool empty = false;
    if (!data_grad) {
        if (!plan_fwd(g, dtype, p, &variant[0])) return false;
        const int n = describe_one(p, variant[0], buf, len);
        const char *note = p.decim ? "; the copy of the input keeps one pixel of every 2 x 2 tile" : !p.tile && fwd_reads_in_place(g, p) ? "; X read in place" : "";
        if (n > 0 && (size_t)n + 1 < len) snprintf(buf + n, len - n, "%s%s", note, record_with_filter(g, p) ? "; the record in the filter's launch" : "");
        return true;
    }
    if (!plan_dx(g, dtype, p, cls, variant, &ncls, &empty)) return false;
    size_t at = 0;
    for (int k = 0; k < ncls && at + 1 < len; ++k) {
        int n = snprintf(buf + at, len - at, "%sclass(%d,%d): ", k ? "; " : "", cls[k].a0, cls[k].b0);
        at += (size_t)max(n, 0);
        if (at + 1 >= len) break;
        n = describe_one(cls[k], variant[k], buf + at, len - at);
        at += (size_t)max(n, 0);
    }
    if (at + 1 < len && dx_reads_in_place(g, cls, ncls) && cls[0].tile != 4) snprintf(buf + at, len - at, "; dY read in place");
    return true;
}

size_t conv_mfma_workspace(const Geom &g, int dtype, bool data_grad)
{
    FwdPlan fwd;
    DxPlan dx;
    if (data_grad) return plan_dx_mfma(g, dtype, &dx) ? dx.ws_bytes : 0;
    return plan_fwd_mfma(g, dtype, &fwd) ? fwd.ws_bytes : 0;
}

// Forward: Y = X * W + b.  False when the geometry is not covered.
bool plan_fwd_mfma(const Geom &g, int dtype, FwdPlan *plan)
{
    if (!plan_fwd(g, dtype, plan->p, &plan->variant)) return false;
    const WsLayout l = fwd_layout(g, plan->p);
    plan->ws_in = l.in;
    plan->ws_wt = l.wt;
    plan->ws_bytes = l.in + l.wt + l.part;
    return true;
}

// *pooled: Z has been written on the way (the channels-last repack reads X anyway); otherwise
// the caller runs the compress kernel.
hipError_t launch_fwd_mfma(const Geom &g, FwdPlan &plan, const void *X, const void *W, const void *b, void *Y, void *Z, void *ws, hipStream_t st,
                           bool *pooled)
{
    GatherParams &p = plan.p;
    hipError_t e = hipSuccess;
    bf16_t *in = (bf16_t *)ws, *wt = (bf16_t *)((char *)ws + plan.ws_in);
    p.part = p.ksplit > 1 ? (float *)((char *)ws + plan.ws_in + plan.ws_wt) : nullptr;
    const bool fuse = Z && record_in_repack(g); // (with `direct` the repack launch forms Z without writing the channels-last copy)
    const bool direct = fwd_reads_in_place(g, p), with_filter = Z && record_with_filter(g, p);
    *pooled = with_filter;
    // nothing to do for the input but the record: the filter's blocks go ahead of the pooling ones in one launch
    const FilterRepack f{(const bf16_t *)W, wt, g.K, g.C, p.ntaps_total, p.Mp, p.KCp, 0};
    if (p.tile == 3) {
        // the input as it lies, the record on the way where the items are row pairs, the filter as it lies where its rows are whole fragments
        if (!p.w_direct) {
            if (with_filter) e = launch_compress_repack(g, X, Z, f, st);
            else e = launch_repack(make_repack(nullptr, in, 0, g.C, g.H * g.W, p.KCp, f.W, wt, g.K, g.C, 1, p.Mp, p.KCp, 0, nullptr, g.W), st);
        }
        if (e != hipSuccess) return e;
        p.in = (const bf16_t *)X;
        p.wt = p.w_direct ? (const bf16_t *)W : wt;
        p.bias = (const bf16_t *)b; p.out = (bf16_t *)Y;
        p.Z = p.pw_pool ? (bf16_t *)Z : nullptr;
        *pooled = *pooled || p.Z;
        return run_gather(p, plan.variant, st);
    }
    if (with_filter) {
        e = launch_compress_repack(g, X, Z, f, st);
    } else {
        e = launch_repack(make_repack((const bf16_t *)X, direct ? nullptr : in, direct && !fuse ? 0 : g.N, g.C, g.H * g.W, p.KCp, f.W, wt,
                                      g.K, g.C, p.ntaps_total, p.Mp, p.KCp, 0, fuse ? (bf16_t *)Z : nullptr, g.W, p.decim), st);
        *pooled = fuse;
    }
    if (e != hipSuccess) return e;
    p.in = direct ? (const bf16_t *)X : in;
    p.nchw = direct;
    p.KCin = g.C;
    p.wt = wt; p.bias = (const bf16_t *)b; p.out = (bf16_t *)Y;
    return run_gather(p, plan.variant, st);
}

// Data gradient: dX = W^T * dY.  False when the geometry is not covered.
bool plan_dx_mfma(const Geom &g, int dtype, DxPlan *plan)
{
    GatherParams base{}, (&cls)[4] = plan->cls;
    plan->empty_class = false;
    if (!plan_dx(g, dtype, base, cls, plan->variant, &plan->ncls, &plan->empty_class)) return false;
    const WsLayout l = dx_layout(g, base, cls, plan->ncls);
    plan->ws_in = l.in;
    plan->ws_wt = l.wt;
    plan->ws_bytes = l.in + l.wt + l.part;
    plan->direct = dx_reads_in_place(g, cls, plan->ncls);
    plan->rep = make_repack(nullptr, nullptr, plan->direct ? 0 : g.N, g.K, g.P * g.Q, base.KCp, nullptr, nullptr, g.K, g.C,
                            base.ntaps_total, base.Mp, base.KCp, 1, nullptr, 0);
    // pixels no output pixel's tap reaches (possible when stride > filter) stay zero
    // (cleared by blocks of a kernel, not by a memset node: callers may capture this call in a HIP graph)
    if (plan->empty_class) plan->rep.zero_n = (long)g.N * g.C * g.H * g.W;
    return true;
}

// The plan's tensors and its part of the workspace.
void bind_dx_mfma(DxPlan *plan, const void *W, const void *dY, void *dX, void *ws)
{
    bf16_t *in = (bf16_t *)ws, *wt = (bf16_t *)((char *)ws + plan->ws_in);
    for (int k = 0; k < plan->ncls; ++k) {
        GatherParams &p = plan->cls[k];
        p.part = p.ksplit > 1 ? (float *)((char *)ws + plan->ws_in + plan->ws_wt) : nullptr;
        p.in = plan->direct ? (const bf16_t *)dY : in;
        p.nchw = plan->direct;
        p.wt = wt; p.bias = nullptr; p.out = (bf16_t *)dX;
    }
    RepackParams &r = plan->rep;
    r.in = (const bf16_t *)dY;
    r.out = in;
    r.f.W = (const bf16_t *)W;
    r.f.Wt = wt;
    r.zero = plan->empty_class ? (bf16_t *)dX : nullptr;
}

// tail: a weight gradient's slice sum, or null.  repacked: plan.rep has run already, in the weight gradient's launch; the sum then
// runs in the first launch of the data gradient, else in that of the repack.
hipError_t launch_dx_mfma(DxPlan &plan, bool repacked, const DwReduceTail *tail, hipStream_t st)
{
    hipError_t e = repacked ? hipSuccess : launch_repack(plan.rep, st, tail);
    if (repacked && tail) plan.cls[0].tail = *tail;
    for (int k = 0; k < plan.ncls && e == hipSuccess; ++k) e = run_gather(plan.cls[k], plan.variant[k], st);
    return e;
}

} // namespace cac
