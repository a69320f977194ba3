// The gather GEMM (conv_gather_kernel) and its launches; what it computes and for whom: conv_mfma.hip, which plans it.  Its kernels are
// compiled in two files, conv_gather.hip and, with a weight gradient's slice sum in the launch, conv_gather_tail.hip.
#pragma once
#include <mutex>

#include "common.h"
#include "conv_mfma.h"
#include "dw_reduce.h"

namespace cac {

namespace {

using gather::KC;
using gather::kMaxItems;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
constexpr uint32_t kNoLoad = 0x80000000u;
constexpr int KCS = gather::KCS;

// ---- the gather GEMM ----------------------------------------------------------------
//
// Workgroup: 4 MFMA waves (WM x WN, a wave owns 64 (m) x 32*NI (pixels)) and 4 copy waves.
// A pixel tile is PT = WN*NI*32 pixels of one image, or IPT whole images when an image has at
// most PT/2 pixels.  The work of a workgroup is a run of "units" (the same tile position in
// consecutive image groups), each unit kbs "stages" of KC input channels (all nkb channel blocks,
// or this workgroup's share of them when several workgroups -- grid z -- share a tile: then the
// epilogue writes float sums for gather_finish_kernel); the stages of the whole run form one
// software pipeline: the copy waves keep two stages of global loads in flight and write the patch
// of stage s+1 into the LDS buffer the MFMA waves are not reading (one barrier per stage).
// Filter fragments come straight from global memory (fragment order, cache resident), fetched
// ahead by the MFMA waves themselves -- six steps with nine taps, eight where taps x channel groups of
// a pass is 4 or 8 (NTT), else two -- whose only
// other memory traffic is LDS reads, so their load counter never waits on the long-latency
// patch loads.
// floor(x / d) with magic = magic_of(d), for the x that divides_exactly allows
__device__ __forceinline__ uint32_t fdiv(uint32_t x, uint32_t magic) { return magic ? __umulhi(x, magic) : x; }
constexpr uint32_t kNoElem = 0x40000000u;

// TR: the accumulators hold the transposed tile (lanes = output channels, registers = pixels):
// a lane then owns runs of 4 consecutive pixels.  Used when consecutive pixels of the launch are
// consecutive and 8-byte aligned in memory; the runs leave as 8-byte stores, or, with
// p.wide_store, through LDS as 16-byte stores that cover whole rows.
// NTT: taps x 32-channel groups of a pass when that is 9 (nine taps, one group), 8 or 4: the operand
// rings described at their declaration; 0: any number of taps, one group, a shallow prefetch.
// TAIL: the launch may have workgroups that add a weight gradient's slices (a form of its own: one workgroup of 90 stages, 1438 -> 53,
// 1 x 1 stride 2 at 6 x 6, batch 7, 33.5 us without the branch, 35.6 with it).
template <int NI, int WM, int WN, bool TR, int NTT, int ITEMS, bool NCHW, bool TAIL>
__global__ void __launch_bounds__(512) conv_gather_kernel(GatherParams p)
{
    constexpr int MI = 2;
    constexpr int PT = WN * NI * 32; // pixel lanes per workgroup
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr bool DEEP = NTT != 0;
    // several groups per pass only in the kernels made for it (constants everywhere else)
    const int t_log2 = (NTT == 4 || NTT == 8) ? p.t_log2 : 0, kcs = (NTT == 4 || NTT == 8) ? p.kcs : KCS;
    const int KCT = KC << t_log2;                   // channels staged per pass
    const uint32_t buf_bytes = (uint32_t)p.patch_px * kcs * 2;

    unsigned bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if constexpr (TAIL) {
        if (!conv_block(p, smem, bx, by, bz)) return;
    }
    const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tau = bx % p.tiles_per_img, run = bx / p.tiles_per_img;
    const int g_begin = run * p.gpw, g_end = min(g_begin + p.gpw, p.ngrp);
    const int kb0 = bz * p.kbs;                     // this workgroup's share of the channel blocks
    const int nstages = (g_end - g_begin) * p.kbs;
    const int ppi = p.Hc * p.Wc;
    const int pix0 = p.IPT > 1 ? 0 : tau * PT;      // first class-grid pixel of the tile
    const int i0 = fdiv(pix0, p.m_wc);               // its row
    // input patch: rows i0*is + dhmin ..., all columns dwmin ... (Wc-1)*is + dwmax
    const int hin0 = i0 * p.is + p.dhmin, win0 = p.dwmin;

    if (wave_id >= 4) {
        // =========================== copy waves ===========================================
        const int tid = threadIdx.x - 256;
        if constexpr (NCHW) {
            // The input in its own layout [N][Cin][Hin][Win] (Win even): an item is 8 channels x 8
            // pixels of one patch row, as in the repack kernel: eight 16-byte loads along the
            // row (4-byte aligned at least), an 8 x 8 transpose in registers, eight 16-byte
            // LDS writes of one pixel's 8 channels each.  Items exist for the image's own
            // columns only; what lies outside the image is zero in both buffers from the start
            // and is never written.  ITEMS here: items per thread (1 or 2).
            const int GX = (p.Win + 7) >> 3;           // 8-pixel groups of an image row
            const int nitems = (p.IPT * p.PH * GX * (KC / 8)) << t_log2;
            uint32_t e0[ITEMS], l0[ITEMS], m8[ITEMS], gq[ITEMS];
            const int co = tid & ((4 << t_log2) - 1);  // channel octet of the stage (256 is a multiple of their number)
#pragma unroll
            for (int q = 0; q < ITEMS; ++q) {
                const int it = tid + 256 * q;
                const int rest = it >> (2 + t_log2);
                const int rows = fdiv(rest, p.m_gx), gx = rest - rows * GX; // (g, pr) as one index
                const int g = fdiv(rows, p.m_ph), pr = rows - g * p.PH;
                const int hin = hin0 + pr, w0 = gx * 8;
                const bool ok = it < nitems && hin >= 0 && hin < p.Hin;
                uint32_t m = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int w = w0 + k;               // written: inside the image and inside the patch
                    if (ok && w < p.Win && w >= win0 && w < win0 + p.PWd) m |= 1u << k;
                }
                m8[q] = m;
                gq[q] = g;
                e0[q] = ok ? (uint32_t)((g * p.KCin + co * 8) * p.Hin + hin) * p.Win + w0 : kNoElem;
                l0[q] = (uint32_t)(((g * p.PH + pr) * p.PWd + (w0 - win0)) * kcs + co * 8) * 2u; // (used under the mask only)
            }
            const rsrc_t rs_in = make_rsrc(p.in, (uint32_t)p.N * p.KCin * p.Hin * p.Win * 2u);
            const uint32_t plane = (uint32_t)p.Hin * p.Win;
            auto fetch = [&](int s, u32x4 (&r)[ITEMS][8]) {
                const int u = fdiv(s, p.m_kbs), kb = kb0 + s - u * p.kbs;
                const int n_base = (g_begin + u) * p.IPT;
                const uint32_t sbase = (uint32_t)(n_base * p.KCin + kb * KCT) * plane;
                const int c_first = kb * KCT + co * 8;   // the item's first channel
                const uint32_t lim = s < nstages ? (uint32_t)max(p.N - n_base, 0) : 0u;
#pragma unroll
                for (int q = 0; q < ITEMS; ++q)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t e = (gq[q] < lim && c_first + i < p.KCin) ? e0[q] + sbase + i * plane : kNoElem;
                        r[q][i] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, e * 2u, 0, 0);
                    }
            };
            auto put = [&](uint32_t buf, const u32x4 (&r)[ITEMS][8]) {
#pragma unroll
                for (int q = 0; q < ITEMS; ++q)
#pragma unroll
                    for (int px = 0; px < 8; ++px) {
                        u32x4 v; // pixel px of the 8 channels: half px%2 of dword px/2 of every row
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const uint32_t lo = r[q][2 * k][px / 2], hi = r[q][2 * k + 1][px / 2];
                            v[k] = (px & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                        }
                        if (m8[q] & (1u << px)) *(u32x4 *)(smem + buf + l0[q] + px * (kcs * 2)) = v;
                    }
            };
            u32x4 ra[ITEMS][8], rb[ITEMS][8];
            fetch(0, ra);
            fetch(1, rb);
            for (uint32_t i = tid; i < 2 * buf_bytes / 16; i += 256) ((u32x4 *)smem)[i] = u32x4{0, 0, 0, 0};
            __syncthreads(); // (the zeros of one thread lie where another writes pixels)
            put(0, ra);
            __syncthreads();
            for (int s = 0; s < nstages; s += 2) {
                fetch(s + 2, ra);
                put(buf_bytes, rb);
                __syncthreads();
                if (s + 1 >= nstages) break;
                fetch(s + 3, rb);
                put(0, ra);
                __syncthreads();
            }
            return;
        }
        const int items = (p.patch_px * (KC / 8)) << t_log2;
        const int v8 = (tid & ((4 << t_log2) - 1)) * 8; // channel offset of this lane's items in the stage
        uint32_t eq[ITEMS], gq[ITEMS], lq[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int it = tid + 256 * q;
            const int pp = it >> (2 + t_log2);
            const int g = fdiv(pp, p.m_img), rem = pp - g * (p.PH * p.PWd);
            const int pr = fdiv(rem, p.m_pwd), pc = rem - pr * p.PWd;
            const int hin = hin0 + pr, win = win0 + pc;
            const bool ok = it < items && hin >= 0 && hin < p.Hin && win >= 0 && win < p.Win;
            eq[q] = ok ? (uint32_t)((g * p.Hin + hin) * p.Win + win) * p.KCp + v8 : kNoElem;
            gq[q] = g;
            lq[q] = it < items ? (uint32_t)(pp * kcs + v8) * 2u : 0xffffffffu;
        }
        const rsrc_t rs_in = make_rsrc(p.in, (uint32_t)p.N * p.Hin * p.Win * p.KCp * 2u);
        // global -> registers for stage s (dead stages load nothing but are issued all the same:
        // the number of loads in flight is then the same on every path)
        auto fetch = [&](int s, u32x4 (&r)[ITEMS]) {
            const int u = fdiv(s, p.m_kbs), kb = kb0 + s - u * p.kbs;
            const int n_base = (g_begin + u) * p.IPT;
            const uint32_t sbase = (uint32_t)n_base * p.Hin * p.Win * p.KCp + kb * KCT;
            const bool lane_ok = s < nstages && kb * KCT + v8 < p.KCp;
            const uint32_t lim = lane_ok ? (uint32_t)max(p.N - n_base, 0) : 0u;
#pragma unroll
            for (int q = 0; q < ITEMS; ++q) {
                const uint32_t e = gq[q] < lim ? eq[q] + sbase : kNoElem;
                r[q] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, e * 2u, 0, 0);
            }
        };
        auto put = [&](uint32_t buf, const u32x4 (&r)[ITEMS]) {
#pragma unroll
            for (int q = 0; q < ITEMS; ++q)
                if (lq[q] != 0xffffffffu) *(u32x4 *)(smem + buf + lq[q]) = r[q];
        };
        u32x4 ra[ITEMS], rb[ITEMS];
        fetch(0, ra);
        fetch(1, rb);
        put(0, ra);
        __syncthreads();
        for (int s = 0; s < nstages; s += 2) {
            // (a stage past the end is written all the same -- zeros into a buffer nobody reads
            // any more -- so that every path consumes every load)
            fetch(s + 2, ra);
            put(buf_bytes, rb);
            __syncthreads();
            if (s + 1 >= nstages) break;
            fetch(s + 3, rb);
            put(0, ra);
            __syncthreads();
        }
        return;
    }

    // =============================== MFMA waves ===========================================
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id;
    const int wm = wave % WM, wn = wave / WM, half = lane >> 5, l32 = lane & 31;
    const int m0 = (by * WM + wm) * 64;            // this wave's first output channel
    const bool wave_live = m0 < p.Mp;              // waves past the (padded) output channels only keep the barriers

    // this lane's pixels: image within the tile, class-grid coordinates, LDS byte offset of their
    // tap-(dhmin,dwmin) input pixel
    uint32_t pbase[NI];
    int pi[NI], pj[NI], pg[NI];
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
        pi[ni] = ok ? i : -1;
        pj[ni] = j;
        pg[ni] = g;
        pbase[ni] = ok ? (uint32_t)(((g * p.PH + (i - i0) * p.is) * p.PWd + j * p.is) * kcs * 2) : 0u;
    }

    f32x16 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[mi][ni][j] = 0.f;

    const rsrc_t rs_w = make_rsrc(p.wt, (uint32_t)p.ntaps_total * p.Mp * p.KCp * 2u);
    const uint32_t kblks = p.KCp / 16, mblks = p.Mp / 32;
    // Per-tap constants in vector registers (uniform values; with constant indices after
    // unrolling they never have to be reloaded inside the loop): byte offset of the tap's
    // filter fragments and LDS byte offset of the tap within the patch (with this half-wave's
    // 8 channels).
    constexpr uint32_t kFrag = 64 * 16; // bytes of one fragment of the repacked filter
    // With T groups of 32 channels per pass, entry tt stands for (tap tt / T, group tt % T): the
    // loops below run over these "taps" and do not know the difference.
    uint32_t wofs[9], toff[9];
    const int ksteps = (KC / 16) << t_log2;         // 16-channel steps of a pass per tap
#pragma unroll
    for (int tt = 0; tt < 9; ++tt) {
        const int t = tt >> t_log2, tb = tt & ((1 << t_log2) - 1);
        wofs[tt] = ((uint32_t)p.wtap[t] * kblks + tb * (KC / 16)) * mblks * kFrag;
        toff[tt] = (uint32_t)(((p.dh[t] - p.dhmin) * p.PWd + (p.dw[t] - p.dwmin)) * kcs + tb * KC + 8 * half) * 2u;
    }
    // this lane's part of a fragment address; a dead wave reads nothing
    const uint32_t wlane = wave_live ? (uint32_t)(m0 >> 5) * kFrag + lane * 16u : kNoLoad;
    // filter fragment of (tap offset wo, 16-channel block kblk) for output channel block mi
    auto wfrag = [&](uint32_t wo, int kblk, int mi) {
        return __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane + wo + (uint32_t)(kblk * mblks + mi) * kFrag, 0, 0);
    };
    // Fragments are fetched two steps ahead: a tap is KC/16 = 2 steps, so while step (t, kk) runs,
    // the fragment of (t+1, kk) -- or of the next stage's first tap -- is requested.  The pixel
    // operands (LDS) are requested one step ahead.
    static_assert(KC / 16 == 2, "the prefetch distance below is one tap");
    u32x4 wcur[MI], wnxt[MI], wnn[MI];
    // DEEP (NTT = 9, 8 or 4 "taps" a pass): a ring of D steps of fragments instead, enough to cover a miss
    // in the vector cache at full MFMA rate.  A stage is 2 * NTT steps, a multiple of D, so that step q of
    // every stage uses ring slot q % D and, once the steps are unrolled, every slot is a fixed
    // register.  The uniform part of a fragment's address goes into the load's scalar offset.
    constexpr int NTTS = DEEP ? NTT : 9;            // (the ring code is compiled, never run, in the kernels without it)
    constexpr int D = NTTS == 9 ? (NI >= 4 ? 3 : 6) : 8, STEPS = NTTS * (KC / 16); // (a step of NI = 4 is twice as long)
    static_assert(STEPS % D == 0, "ring slots must not move from stage to stage");
    u32x4 wr[DEEP ? D : 1][MI];
    uint32_t wl[9];
    if constexpr (DEEP) {
#pragma unroll
        for (int t = 0; t < 9; ++t) wl[t] = wlane + wofs[t];
#pragma unroll
        for (int q = 0; q < D; ++q)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                wr[q][mi] = __builtin_amdgcn_raw_buffer_load_b128(
                    rs_w, wl[q >> 1], (uint32_t)((kb0 * ksteps + (q & 1)) * mblks + mi) * kFrag, 0);
    } else {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            wcur[mi] = wfrag(wofs[0], kb0 * ksteps, mi);
            wnxt[mi] = wfrag(wofs[0], kb0 * ksteps + 1, mi);
        }
    }

    // TR epilogues: a lane's output channels are fixed, so their bias is fetched here, once, and
    // not in the epilogue, where the load's latency would lie bare
    float bias_tr[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int m = m0 + mi * 32 + l32;
        bias_tr[mi] = (TR && p.bias && m < p.M) ? bf16_to_f32(p.bias[m]) : 0.f;
    }

    if constexpr (NCHW) __syncthreads(); // the copy waves have zeroed both buffers
    __syncthreads(); // buffer 0 holds stage 0
    int kb = 0, unit = 0;
    for (int s = 0; s < nstages; ++s) {
        if (wave_live) {
            const uint32_t buf = (s & 1) ? buf_bytes : 0u;
            const int kb_next = kb + 1 == p.kbs ? 0 : kb + 1;
            u32x4 bcur[NI], bnxt[NI];
            if constexpr (!DEEP) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) bcur[ni] = *(const u32x4 *)(smem + buf + pbase[ni] + toff[0]);
            }
            if constexpr (DEEP) {
                const uint32_t so_cur = (uint32_t)((kb0 + kb) * ksteps * mblks) * kFrag;
                const uint32_t so_nxt = (uint32_t)((kb0 + kb_next) * ksteps * mblks) * kFrag;
                // pixel operands: a ring of DB steps in registers of their own (a copy from a
                // "next" to a "current" set lets the compiler merge the two and issue the LDS read
                // only after the current value's last use, a fraction of a step ahead)
                constexpr int DB = (NI >= 4 || NTTS != 9) ? 2 : 3;
                static_assert(STEPS % DB == 0, "ring slots must not move from stage to stage");
                u32x4 bq[DB][NI];
                auto pixels = [&](int q, int ni) { return *(const u32x4 *)(smem + buf + pbase[ni] + toff[q >> 1] + 32 * (q & 1)); };
#pragma unroll
                for (int q = 0; q < DB - 1; ++q)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) bq[q][ni] = pixels(q, ni);
#pragma unroll
                for (int q = 0; q < STEPS; ++q) {
                    // pixels of step q + DB - 1 (nothing past the stage's last step: the other
                    // buffer is not ready yet)
                    if (q + DB - 1 < STEPS) {
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) bq[(q + DB - 1) % DB][ni] = pixels(q + DB - 1, ni);
                    }
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int mi = 0; mi < MI; ++mi) {
                            union { u32x4 u; bf16x8 v; } af, bf;
                            af.u = wr[q % D][mi];
                            bf.u = bq[q % DB][ni];
                            acc[mi][ni] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf.v, af.v, acc[mi][ni], 0, 0, 0)
                                             : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af.v, bf.v, acc[mi][ni], 0, 0, 0);
                        }
                    // refill the slot with the fragments of step q + D (of this stage or the next;
                    // after the last stage: of the first again, never used)
                    const int q2 = q + D < STEPS ? q + D : q + D - STEPS;
                    const uint32_t so = (q + D < STEPS ? so_cur : so_nxt) + (uint32_t)((q2 & 1) * mblks) * kFrag;
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
                        wr[q % D][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wl[q2 >> 1], so + mi * kFrag, 0);
                    // Pin the order LDS reads, MFMAs, refill, and keep the instruction scheduler from
                    // moving anything to another step (it would sink the loads towards their uses).
                    // one LDS read or one filter load after each MFMA, in its shadow
                    if (q + DB - 1 < STEPS) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, NI - 1, 0);
                    } else {
                        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, MI * NI - 3, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, MI - 1, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                if (t >= p.ntaps) break;
                const bool last = t + 1 >= p.ntaps;
                const uint32_t wo_n = last ? wofs[0] : wofs[t + 1 < 9 ? t + 1 : 0];
                const uint32_t to_n = toff[t + 1 < 9 ? t + 1 : 0];
                const int kblk_n = (kb0 + (last ? kb_next : kb)) * ksteps;
#pragma unroll
                for (int kk = 0; kk < KC / 16; ++kk) {
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) wnn[mi] = wfrag(wo_n, kblk_n + kk, mi);
                    // next step's pixels: the second channel half of this tap, or the next tap
                    // (nothing after the stage's last step: the other buffer is not ready yet)
                    if (kk == 0) {
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) bnxt[ni] = *(const u32x4 *)(smem + buf + pbase[ni] + toff[t] + 32);
                    } else if (!last) {
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) bnxt[ni] = *(const u32x4 *)(smem + buf + pbase[ni] + to_n);
                    }
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int mi = 0; mi < MI; ++mi) {
                            union { u32x4 u; bf16x8 v; } af, bf;
                            af.u = wcur[mi];
                            bf.u = bcur[ni];
                            acc[mi][ni] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf.v, af.v, acc[mi][ni], 0, 0, 0)
                                             : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af.v, bf.v, acc[mi][ni], 0, 0, 0);
                        }
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) {
                        wcur[mi] = wnxt[mi];
                        wnxt[mi] = wnn[mi];
                    }
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) bcur[ni] = bnxt[ni];
                }
            }
            if (kb == p.kbs - 1) {
                // ---- epilogue of the unit: bias, bfloat16, NCHW
                const int n_base = (g_begin + unit) * p.IPT;
                if (TR && p.wide_store) {
                    // Through LDS (a region of the wave's own, past the staging buffers), so that
                    // the lanes of a store cover whole rows: the wave's 64 channels x NI*32 pixels
                    // as [channel][pixel] bfloat16, rows padded by 16 bytes; then 8 pixels (16 bytes)
                    // per lane, NI*4 neighbouring lanes one channel's run.
                    // Two pixel blocks (64 pixels) per pass, so that the region stays at 9 KB per wave.
                    constexpr int NIB = NI < 2 ? NI : 2, ROWB = NIB * 64 + 16, LPR = NIB * 4;
                    unsigned char *ep = smem + 2 * buf_bytes + wave * (64 * ROWB);
                    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
#pragma unroll
                    for (int pass = 0; pass < NI / NIB; ++pass) {
#pragma unroll
                        for (int mi = 0; mi < MI; ++mi) {
                            const float bias = bias_tr[mi];
#pragma unroll
                            for (int nb = 0; nb < NIB; ++nb)
#pragma unroll
                                for (int jq = 0; jq < 4; ++jq) {
                                    const f32x16 &a = acc[mi][pass * NIB + nb];
                                    *(u32x2 *)(ep + (mi * 32 + l32) * ROWB + (nb * 32 + 8 * jq + 4 * half) * 2) =
                                        u32x2{f32x2_to_bf16x2(a[4 * jq] + bias, a[4 * jq + 1] + bias), f32x2_to_bf16x2(a[4 * jq + 2] + bias, a[4 * jq + 3] + bias)};
                                }
                        }
                        // (the wave reads what it wrote itself: LDS serves a wave's requests in order)
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                        const int seg = lane % LPR, idx = (wn * NI + pass * NIB) * 32 + seg * 8; // pixel of the tile
                        int g = 0, px = pix0 + idx;
                        if (p.IPT > 1) {
                            g = fdiv(idx, p.m_ppi);
                            px = idx - g * ppi;
                        }
                        const int n = n_base + g;
                        const bool px_ok = px < ppi && g < p.IPT && n < p.N;
#pragma unroll
                        for (int it = 0; it < LPR; ++it) {
                            const int row = it * (64 / LPR) + lane / LPR, m = m0 + row;
                            const u32x4 v = *(const u32x4 *)(ep + row * ROWB + seg * 16);
                            if (px_ok && m < p.M) *(u32x4 *)(p.out + ((long)n * p.M + m) * ppi + px) = v;
                        }
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                    }
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                            for (int j = 0; j < 16; ++j) acc[mi][ni][j] = 0.f;
                } else if constexpr (TR) {
                    // register j of lane l: pixel 8*(j/4) + 4*(l/32) + j%4 of the block, channel l%32
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) {
                        const int m = m0 + mi * 32 + l32;
                        const float bias = bias_tr[mi];
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                            for (int jq = 0; jq < 4; ++jq) {
                                // the 4 pixels idx .. idx+3 of the tile (same image: an image's pixel
                                // count is a multiple of 4 on this path)
                                const int idx = (wn * NI + ni) * 32 + 8 * jq + 4 * half;
                                int g = 0, px = pix0 + idx;
                                if (p.IPT > 1) {
                                    g = fdiv(idx, p.m_ppi);
                                    px = idx - g * ppi;
                                }
                                const int n = n_base + g;
                                if (m < p.M && px < ppi && g < p.IPT && n < p.N) {
                                    const f32x16 &a = acc[mi][ni];
                                    if (p.part) { // a share of the channels: float sums, finished by gather_finish_kernel
                                        typedef __attribute__((ext_vector_type(4))) float f32x4;
                                        *(f32x4 *)(p.part + (((long)bz * p.N + n) * p.M + m) * ppi + px) =
                                            f32x4{a[4 * jq], a[4 * jq + 1], a[4 * jq + 2], a[4 * jq + 3]};
                                        continue;
                                    }
                                    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
                                    const u32x2 v = {f32x2_to_bf16x2(a[4 * jq] + bias, a[4 * jq + 1] + bias), f32x2_to_bf16x2(a[4 * jq + 2] + bias, a[4 * jq + 3] + bias)};
                                    *(u32x2 *)(p.out + ((long)n * p.M + m) * ppi + px) = v;
                                }
                            }
                    }
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                            for (int j = 0; j < 16; ++j) acc[mi][ni][j] = 0.f;
                } else {
                    // register j of lane l: channel 8*(j/4) + 4*(l/32) + j%4, pixel l%32 of the block
                    // Stores through a buffer descriptor over the whole output (less than 2^31 bytes on this
                    // path): 32-bit offsets, split into the pixel's part (per block) and the channel's, and
                    // an offset past the tensor instead of a branch for lanes that own no output.
                    const rsrc_t rs_out = make_rsrc(p.out, (uint32_t)p.N * p.M * p.Hout * p.Wout * 2u);
                    const uint32_t plane_out = (uint32_t)p.Hout * p.Wout;
                    uint32_t obase[NI];
                    bool oky[NI];
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        const int n = n_base + pg[ni];
                        const int h = pi[ni] * p.os + p.a0, w = pj[ni] * p.os + p.b0;
                        oky[ni] = pi[ni] >= 0 && n < p.N;
                        obase[ni] = oky[ni] ? ((uint32_t)n * p.M * plane_out + h * p.Wout + w) * 2u : 0u;
                    }
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                        for (int j = 0; j < 16; ++j) {
                            const int m = m0 + mi * 32 + 8 * (j / 4) + 4 * half + (j % 4);
                            const float bias = (p.bias && m < p.M) ? bf16_to_f32(p.bias[m]) : 0.f;
                            const uint32_t moff = (uint32_t)min(m, p.M) * plane_out * 2u;
#pragma unroll
                            for (int ni = 0; ni < NI; ++ni) {
                                const uint32_t off = (m < p.M && oky[ni]) ? obase[ni] + moff : kNoLoad;
                                __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(acc[mi][ni][j] + bias), rs_out, off, 0, 0);
                                acc[mi][ni][j] = 0.f;
                            }
                        }
                }
            }
        }
        if (++kb == p.kbs) {
            kb = 0;
            ++unit;
        }
        __syncthreads();
    }
}

// out = bfloat16(bias + sum over the channel shares of their float sums), 4 pixels per thread.
__global__ void __launch_bounds__(256) gather_finish_kernel(const float *__restrict__ part, const bf16_t *__restrict__ bias,
                                                            bf16_t *__restrict__ out, long quads, int nsplit, int ppi, int M)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
    const long q = (long)blockIdx.x * 256 + threadIdx.x;
    if (q >= quads) return;
    const f32x4 *src = (const f32x4 *)part + q;
    f32x4 sum = src[0];
    for (int k = 1; k < nsplit; ++k) sum += src[k * quads];
    if (bias) sum += bf16_to_f32(bias[((uint32_t)q * 4u / (uint32_t)ppi) % (uint32_t)M]); // (fewer than 2^30 quads)
    const u32x2 v = {f32x2_to_bf16x2(sum[0], sum[1]), f32x2_to_bf16x2(sum[2], sum[3])};
    *((u32x2 *)out + q) = v;
}

template <int NI, int WM, int WN, bool TR, int NTT, int ITEMS, bool NCHW, bool TAIL> hipError_t launch_gather_items(const GatherParams &p, hipStream_t st)
{
    auto kern = conv_gather_kernel<NI, WM, WN, TR, NTT, ITEMS, NCHW, TAIL>;
    // (per instantiation; once per process, whichever host thread comes first)
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    const int runs = (p.ngrp + p.gpw - 1) / p.gpw;
    dim3 grid(p.tiles_per_img * runs, (p.Mp / 64 + WM - 1) / WM, p.ksplit);
    const size_t lds = max((size_t)2 * p.patch_px * p.kcs * 2, (size_t)(TAIL ? 8192 : 0)) + (p.wide_store ? 4 * 64 * ((NI < 2 ? NI : 2) * 64 + 16) : 0);
    GatherParams q = p;
    grid = share_grid(q, grid, 512);
    hipLaunchKernelGGL(kern, grid, dim3(512), lds, st, q);
    if (p.ksplit > 1) {
        const long quads = (long)p.N * p.M * p.Hc * p.Wc / 4;
        hipLaunchKernelGGL(gather_finish_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, (const float *)p.part,
                           p.bias, p.out, quads, p.ksplit, p.Hc * p.Wc, p.M);
    }
    return hipGetLastError();
}

// (small patches: half the items, half the loads per stage and a shorter start-up)
template <int NI, int WM, int WN, bool TR, int NTT, bool TAIL> hipError_t launch_gather_shape(const GatherParams &p, hipStream_t st)
{
    if (p.nchw) // items of 8 x 8 elements, one or two per copy thread
        return p.IPT * p.PH * ((p.Win + 7) / 8) * (KC / 8) * p.T <= 256 ? launch_gather_items<NI, WM, WN, TR, NTT, 1, true, TAIL>(p, st)
                                                                         : launch_gather_items<NI, WM, WN, TR, NTT, 2, true, TAIL>(p, st);
    return p.patch_px * (KC / 8) * p.T <= 256 * 6 ? launch_gather_items<NI, WM, WN, TR, NTT, 6, false, TAIL>(p, st)
                                                  : launch_gather_items<NI, WM, WN, TR, NTT, kMaxItems, false, TAIL>(p, st);
}

template <int NI, int WM, int WN, bool TAIL> hipError_t launch_gather(const GatherParams &p, hipStream_t st)
{
    // runs of 4 pixels are contiguous and 8-byte aligned: the class grid is the whole output
    // plane and a plane is a multiple of 4 pixels
    const bool packed = p.os == 1 && p.Hc == p.Hout && p.Wc == p.Wout && (p.Hc * p.Wc) % 4 == 0;
    // (the planner gives T > 1 only where taps x T is 4 or 8)
    const int ntt = p.ntaps * p.T;
    if (ntt == 9 && p.T == 1) return packed ? launch_gather_shape<NI, WM, WN, true, 9, TAIL>(p, st) : launch_gather_shape<NI, WM, WN, false, 9, TAIL>(p, st);
    if (ntt == 8) return packed ? launch_gather_shape<NI, WM, WN, true, 8, TAIL>(p, st) : launch_gather_shape<NI, WM, WN, false, 8, TAIL>(p, st);
    if (ntt == 4) return packed ? launch_gather_shape<NI, WM, WN, true, 4, TAIL>(p, st) : launch_gather_shape<NI, WM, WN, false, 4, TAIL>(p, st);
    if (p.T != 1) return hipErrorInvalidValue; // (never planned)
    return packed ? launch_gather_shape<NI, WM, WN, true, 0, TAIL>(p, st) : launch_gather_shape<NI, WM, WN, false, 0, TAIL>(p, st);
}

template <bool TAIL> hipError_t launch_gather_variant(const GatherParams &p, int variant, hipStream_t st)
{
    switch (variant) {
    case 0: return launch_gather<2, 1, 4, TAIL>(p, st);
    case 1: return launch_gather<2, 2, 2, TAIL>(p, st);
    case 2: return launch_gather<2, 4, 1, TAIL>(p, st);
    case 3: return launch_gather<1, 1, 4, TAIL>(p, st);
    case 4: return launch_gather<1, 2, 2, TAIL>(p, st);
    default: return launch_gather<1, 4, 1, TAIL>(p, st);
    }
}

} // namespace

} // namespace cac
