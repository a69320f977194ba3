// Nine-tap gather GEMM (3 x 3 forward convolution and data gradient, stride 1 or 2) for layers with few pixels: every wave stages
// for itself, the waves of a workgroup share a tile's channels.
//
// The sum is the one of conv_mfma.hip, filter fragments and taps as there.  Where pixels are few, what bounds the other
// kernels is latency: a barrier between any two stages, one workgroup or less to a compute unit, a channels-last copy of the
// input in front and, with the channels shared out over workgroups, a launch behind that adds float sums.  Here
//   - a tile is 32 * MI output channels x 64 pixels, pixels running on from image to image (maps of 25, 36 or 49 pixels
//     leave no lane idle), and its KS waves take every KS-th stage of KC channels each: no barrier stands between two
//     stages, the waves of a compute unit are at different points and fill each other's gaps; their sums meet once, in LDS,
//     in wave order;
//   - a wave stages the rows that its tile reaches in LDS of its own, from the tensor as it lies (rows of any length);
//     halo rows and columns are zeros from the start and never written;
//   - filter fragments come from global memory, D steps ahead in registers, no two waves of a workgroup the same ones; an
//     XCD works on all pixel tiles of one block of output channels after the other, so that its L2 keeps the filter.
// Measured per call (repack launch included): 512 -> 512 at 4 x 4, batch 128, a step 71 -> 60 us; long sums for few tiles, 1380 -> 32
// at 5 x 5, batch 1: 69 -> 19; 528 -> 388 at 7 x 7, batch 42, data gradient: 40 -> 22 (conv_tile.hip).  In the mean over random
// layers 0.59 of the gather's time.  Up to 256 registers (none spilled) bound the waves, two to a SIMD; filter fragments are what a compute unit
// asks L2 for: 1 KiB per wave and two MFMAs.
#include <stdio.h>
#include <stdlib.h>

#include <mutex>

#include "common.h"
#include "conv_mfma.h"
#include "tile_stage.h"
#include "wave_rows.h"

namespace cac {

namespace {

using namespace tile;
constexpr int TAPS = 9, NI = 2, PT = 32 * NI; // pixels of a tile
constexpr int kOutRow = PT * 2 + 16;          // LDS bytes of an output row: a channel's pixels
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) f32x4 *lds_f32x4_ptr;

__device__ __forceinline__ WaveRows rows_of(const GatherParams &p) { return WaveRows{p.VH, p.PH, p.IR}; }

constexpr int red_bytes(int MI, int KS) { return (KS - 1) * MI * NI * 4 * 1024; }

// (a wave reads what it wrote itself: LDS serves a wave's requests in order)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's staging: KC channels of the rows that its tile reaches, in LDS as [pixel][KC + 8].  An item is 8 channels x GW pixels of
// one row (8; 7 in rows of odd length, read from the dword below an odd element); a lane has ITEMS of them.
template <int KC, int ITEMS, int GW> struct WaveStage {
    static constexpr int KCS = KC + 8, OCT = KC / 8;
    uint32_t e0[ITEMS], l0[ITEMS], m8[ITEMS], dump;
    u32x4 r[ITEMS][8];
    int co, K, nkb, plane;
    rsrc_t rs_in;

    // rows of the images from the first one the tile reaches on, one after the other
    __device__ __forceinline__ void init(const GatherParams &p, uint32_t wbase, uint32_t dump_at, int n0, int i0)
    {
        const int lane = threadIdx.x & 63, hfirst = wave_first_row(i0, p.is, p.dhmin, p.Hin);
        const WaveRows rows = rows_of(p);
        co = lane & (OCT - 1);
        K = p.KCin;
        nkb = p.nkb;
        plane = p.Hin * p.Win;
        dump = dump_at;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int it = lane + 64 * q, rest = it / OCT;
            const int row = fdiv(rest, p.m_gx), gx = rest - row * p.GX;
            const int gi = fdiv(hfirst + row, p.m_ph), w0 = gx * GW;
            const WaveRow at = wave_row(rows, p.Hin, p.is, p.dhmin, i0, hfirst, row, gi);
            const bool ok = at.ok & (n0 + gi < p.N);
            uint32_t m = 0;
#pragma unroll
            for (int k = 0; k < GW; ++k) {
                const int w = w0 + k;
                m |= (ok & (w < p.Win) & (w >= p.dwmin) & (w < p.dwmin + p.PWd)) ? 1u << k : 0u;
            }
            m8[q] = m;
            e0[q] = ok ? (uint32_t)(((n0 + gi) * K + co * 8) * p.Hin + at.hin) * p.Win + w0 : kNoElem;
            l0[q] = wbase + (uint32_t)((at.lr * p.PWd + (w0 - p.dwmin)) * KCS + co * 8) * 2u;
        }
        rs_in = make_rsrc(p.in, (uint32_t)p.N * K * plane * 2u);
    }
    __device__ __forceinline__ void clear(uint32_t wbase, uint32_t bytes)
    {
        for (uint32_t i = threadIdx.x & 63; i < bytes / 16; i += 64) *(lds_u32x4_ptr)(uintptr_t)(wbase + 16 * i) = u32x4{0, 0, 0, 0};
        wave_sync();
    }
    __device__ __forceinline__ void fetch(int s)
    {
        const uint32_t sbase = (uint32_t)(s * KC) * plane;
        const int nvalid = s < nkb ? K - (s * KC + co * 8) : 0; // channels that exist
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            uint32_t e = e0[q] + sbase; // (no item: still far outside the tensor)
            opaque(e);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t ei = i < nvalid ? e : kNoElem;
                r[q][i] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, (GW == 7 ? ei & ~1u : ei) * 2u, 0, 0);
                e += plane;
            }
        }
    }
    __device__ __forceinline__ void put(int s)
    {
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            if constexpr (GW == 7) { // (read from the dword below an odd element: down by one)
                const uint32_t par = e0[q] + (uint32_t)(s * KC) * plane;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t sh = ((par + i * plane) & 1u) * 16u;
#pragma unroll
                    for (int k = 0; k < 3; ++k) r[q][i][k] = __builtin_amdgcn_alignbit(r[q][i][k + 1], r[q][i][k], sh);
                    r[q][i][3] >>= sh;
                }
            }
#pragma unroll
            for (int px = 0; px < GW; ++px) {
                u32x4 x; // pixel px of the 8 channels
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t lo = r[q][2 * k][px / 2], hi = r[q][2 * k + 1][px / 2];
                    x[k] = (px & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                }
                // (a pixel that is not wanted goes to a place of the lane's own past the buffers: no branch)
                *(lds_u32x4_ptr)(uintptr_t)((m8[q] & (1u << px)) ? l0[q] + px * (KCS * 2) : dump) = x;
            }
        }
    }
};

// ITEMS: 8 channels x GW pixels that a lane stages per stage.
template <int MI, int KC, int ITEMS, int GW, int KS> __global__ void __launch_bounds__(64 * KS, 2) conv_wave_kernel(GatherParams p)
{
    constexpr int KSTEPS = KC / 16, STEPS = TAPS * KSTEPS, KCS = KC + 8;
    constexpr int D = 9; // steps of filter fragments in flight
    static_assert(STEPS % D == 0, "ring slots must not move from stage to stage");
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned bx, by, bz;
    if (!conv_block(p, smem, bx, by, bz)) return;
    const int per_xcd = p.gx >> 3, v = (bx & 7) * per_xcd + (bx >> 3);
    if (v >= p.tiles_per_img * p.mtiles) return; // (tiles_per_img: pixel tiles of all images)
    const int mt = v / p.tiles_per_img, m0 = mt * 32 * MI, F = (v - mt * p.tiles_per_img) * PT; // first pixel, over all images
    const int ppi = p.Hc * p.Wc, nkb = p.nkb;
    const int n0 = F / ppi, px0 = F - n0 * ppi, i0 = fdiv(px0, p.m_wc);

    WaveStage<KC, ITEMS, GW> in;
    const uint32_t wbase = lds0 + ks * p.buf_bytes;
    in.init(p, wbase, lds0 + KS * p.buf_bytes + threadIdx.x * 16, n0, i0);

    const rsrc_t rs_w = make_rsrc(p.wt, (uint32_t)TAPS * p.Mp * p.KCp * 2u);
    const uint32_t kstep = (p.Mp / 32) * kFrag, wlane = (uint32_t)(mt * MI) * kFrag + lane * 16u;
    f32x16 acc[NI][MI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[ni][mi][j] = 0.f;
    u32x4 wr[D][MI];
    if (ks < nkb) {
        in.fetch(ks);
#pragma unroll
        for (int q = 0; q < D; ++q)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                wr[q][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, p.wofs[q / KSTEPS] + (ks * KSTEPS + q % KSTEPS) * kstep + mi * kFrag, 0);
    }
    float bias[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int m = m0 + mi * 32 + l32;
        bias[mi] = (p.bias && m < p.M) ? bf16_to_f32(p.bias[m]) : 0.f;
    }
    // ---- this lane's pixels
    uint32_t pbase[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int f = px0 + ni * 32 + l32;
        const int gi = fdiv(f, p.m_ppi), px = f - gi * ppi, i = fdiv(px, p.m_wc), j = px - i * p.Wc;
        const uint32_t at = (uint32_t)((wave_pixel_row(rows_of(p), p.is, i0, gi, i) * p.PWd + j * p.is) * KCS * 2);
        pbase[ni] = wbase + 16u * half + (n0 + gi < p.N ? at : 0u);
    }
    in.clear(wbase, p.buf_bytes);

    for (int s = ks; s < nkb; s += KS) {
        in.put(s);
        wave_sync();
        in.fetch(s + KS); // (past the end: nothing is loaded)
        uint32_t so = (uint32_t)s * KSTEPS * kstep, so_next = (uint32_t)wave_next_stage(s, KS, nkb) * KSTEPS * kstep;
        opaque_s(so);
        opaque_s(so_next);
        u32x4 bq[2][NI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) bq[0][ni] = lds16(pbase[ni] + p.toff[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < STEPS; ++q) {
            if (q + 1 < STEPS) {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) bq[(q + 1) & 1][ni] = lds16(pbase[ni] + p.toff[(q + 1) / KSTEPS] + 32 * ((q + 1) % KSTEPS));
            }
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) {
                    union { u32x4 u; bf16x8 v; } af, bf;
                    af.u = wr[q % D][mi];
                    bf.u = bq[q & 1][ni];
                    acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf.v, af.v, acc[ni][mi], 0, 0, 0);
                }
            // refill the ring with the fragments of step q + D
            const int q2 = q + D < STEPS ? q + D : q + D - STEPS;
            const uint32_t so2 = p.wofs[q2 / KSTEPS] + (q + D < STEPS ? so : so_next) + q2 % KSTEPS * kstep;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) wr[q % D][mi] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, so2 + mi * kFrag, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        wave_sync();
    }

    // ---- the sums of the KS waves, in groups of four pixels: wave ks finishes groups [ks * GK, (ks + 1) * GK) and is handed
    // the others' parts of them, red[finishing wave][source wave, itself left out][group][lane]
    constexpr int G = NI * MI * 4, GK = G / KS;
    static_assert(G % KS == 0, "");
    const uint32_t out = lds0 + red_bytes(MI, KS); // [channel][pixel], bfloat16
    __syncthreads(); // (all staging buffers are dead)
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int dst = g / GK;
        const f32x16 &a = acc[g / (MI * 4)][g / 4 % MI];
        if (dst != ks)
            *(lds_f32x4_ptr)(uintptr_t)(lds0 + (uint32_t)(((dst * (KS - 1) + (ks < dst ? ks : ks - 1)) * GK + g % GK) * 1024) + lane * 16) =
                f32x4{a[4 * (g % 4)], a[4 * (g % 4) + 1], a[4 * (g % 4) + 2], a[4 * (g % 4) + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (g / GK != ks) continue;
        const int ni = g / (MI * 4), mi = g / 4 % MI, jq = g % 4;
        const f32x16 &a = acc[ni][mi];
        f32x4 sum;
#pragma unroll
        for (int src = 0; src < KS; ++src) {
            f32x4 t = f32x4{a[4 * jq], a[4 * jq + 1], a[4 * jq + 2], a[4 * jq + 3]};
            if (src != ks) t = *(lds_f32x4_ptr)(uintptr_t)(lds0 + (uint32_t)(((ks * (KS - 1) + (src < ks ? src : src - 1)) * GK + g % GK) * 1024) + lane * 16);
            if (src == 0) sum = t;
            else sum += t;
        }
        *(lds_u32x2_ptr)(uintptr_t)(out + (uint32_t)((mi * 32 + l32) * kOutRow + (ni * 32 + 8 * jq + 4 * half) * 2)) =
            u32x2{f32x2_to_bf16x2(sum[0] + bias[mi], sum[1] + bias[mi]), f32x2_to_bf16x2(sum[2] + bias[mi], sum[3] + bias[mi])};
    }
    __syncthreads();
    // ---- rows of the tile to memory, V pixels (of one image: V divides its pixels) per lane
    const rsrc_t rs_out = make_rsrc(p.out, (uint32_t)p.N * p.M * ppi * 2u);
    auto store = [&](auto vtag) {
        constexpr int V = decltype(vtag)::value, LPR = PT / V, RPI = 64 * KS / LPR; // lanes of a row; rows at a time
        const int seg = threadIdx.x % LPR, row0 = threadIdx.x / LPR, f = px0 + seg * V;
        const int gi = fdiv(f, p.m_ppi), px = f - gi * ppi, n = n0 + gi;
        const uint32_t base = (uint32_t)(n * p.M + m0) * ppi + px;
#pragma unroll
        for (int it = 0; it < (32 * MI + RPI - 1) / RPI; ++it) {
            const int row = it * RPI + row0;
            const uint32_t off = ((row < 32 * MI) & (n < p.N) & (m0 + row < p.M)) ? (base + (uint32_t)row * ppi) * 2u : kNoLoad;
            const uint32_t src = out + (row < 32 * MI ? row : 0) * kOutRow + seg * (V * 2);
            if constexpr (V == 8) __builtin_amdgcn_raw_buffer_store_b128(lds16(src), rs_out, off, 0, 0);
            else if constexpr (V == 4) __builtin_amdgcn_raw_buffer_store_b64(*(lds_u32x2_ptr)(uintptr_t)src, rs_out, off, 0, 0);
            else if constexpr (V == 2) __builtin_amdgcn_raw_buffer_store_b32(*(lds_u32_ptr)(uintptr_t)src, rs_out, off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b16(*(lds_u16_ptr)(uintptr_t)src, rs_out, off, 0, 0);
        }
    };
    if (p.store_px == 8) store(std::integral_constant<int, 8>{});
    else if (p.store_px == 4) store(std::integral_constant<int, 4>{});
    else if (p.store_px == 2) store(std::integral_constant<int, 2>{});
    else store(std::integral_constant<int, 1>{});
}

// The 3 x 3 stride-2 data gradient, padding 1: all parity classes of dX in one launch.  Pixel (2i + a, 2j + b) has the taps with r = 1 (a = 0)
// or r = 0, 2 (a = 1), s likewise, of dY at (i + (r == 0), j + (s == 0)): a step of 16 channels is nine products for every block of 32
// pixels of dY, over four shifts of it.  A tile is 32 input channels x 32 * BL pixels of dY x 4 classes; the two classes of a row of dX
// leave side by side.  128 accumulators and nine filter fragments ahead make 2 waves to a SIMD; what bounds it is the wait for a
// stage.  Per call: 69 input and 1472 output channels at 26 x 49, batch 30, 154 -> 49 us against four launches of the gather;
// 423 and 408 at 13 x 13, batch 2, 53 -> 14.5; over 158 random layers (odd rows) 0.35 of its time, none slower.  Against conv_dx2.hip:
// 44 and 1888 at 6 x 6, batch 125, 93 -> 26 us.
constexpr int kPairRow(int BL) { return 32 * BL * 4 + 16; } // LDS bytes of a channel's pairs of pixels
constexpr int red2_bytes(int BL, int KS) { return (KS - 1) * 2 * BL * 4 * 1024; }

template <int BL, int KC, int GW, int KS> __global__ void __launch_bounds__(64 * KS, 2) conv_wave_dx2_kernel(GatherParams p)
{
    constexpr int KSTEPS = KC / 16, KCS = KC + 8, PT = 32 * BL;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    unsigned bx, by, bz;
    if (!conv_block(p, smem, bx, by, bz)) return;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_xcd = p.gx >> 3, v = (bx & 7) * per_xcd + (bx >> 3);
    if (v >= p.tiles_per_img * p.mtiles) return;
    const int mt = v / p.tiles_per_img, m0 = mt * 32, F = (v - mt * p.tiles_per_img) * PT;
    const int ppi = p.Hc * p.Wc, nkb = p.nkb;
    const int n0 = F / ppi, px0 = F - n0 * ppi, i0 = fdiv(px0, p.m_wc);
    WaveStage<KC, 1, GW> in;
    const uint32_t wbase = lds0 + ks * p.buf_bytes;
    in.init(p, wbase, lds0 + KS * p.buf_bytes + threadIdx.x * 16, n0, i0);
    const rsrc_t rs_w = make_rsrc(p.wt, (uint32_t)TAPS * p.Mp * p.KCp * 2u);
    const uint32_t kstep = (p.Mp / 32) * kFrag, wlane = (uint32_t)mt * kFrag + lane * 16u;
    // class 2 * a + b of a tap, and its shift of dY, 2 * (r == 0) + (s == 0)
    constexpr auto cls = [](int t) { return 2 * (t / 3 != 1) + (t % 3 != 1); };
    constexpr auto shift = [](int t) { return 2 * (t / 3 == 0) + (t % 3 == 0); };
    f32x16 acc[4][BL];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int bl = 0; bl < BL; ++bl)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[c][bl][j] = 0.f;
    u32x4 wr[TAPS];
    if (ks < nkb) {
        in.fetch(ks);
#pragma unroll
        for (int t = 0; t < TAPS; ++t) wr[t] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, p.wofs[t] + ks * KSTEPS * kstep, 0);
    }
    uint32_t pbase[BL];
#pragma unroll
    for (int bl = 0; bl < BL; ++bl) {
        const int f = px0 + bl * 32 + l32;
        const int gi = fdiv(f, p.m_ppi), px = f - gi * ppi, i = fdiv(px, p.m_wc), j = px - i * p.Wc;
        pbase[bl] = wbase + 16u * half + (n0 + gi < p.N ? (uint32_t)((wave_pixel_row(rows_of(p), 1, i0, gi, i) * p.PWd + j) * KCS * 2) : 0u);
    }
    in.clear(wbase, p.buf_bytes);
    for (int s = ks; s < nkb; s += KS) {
        in.put(s);
        wave_sync();
        in.fetch(s + KS); // (past the end: nothing is loaded)
        uint32_t so = (uint32_t)s * KSTEPS * kstep, so_next = (uint32_t)wave_next_stage(s, KS, nkb) * KSTEPS * kstep;
        opaque_s(so);
        opaque_s(so_next);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            u32x4 bq[4][BL];
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int bl = 0; bl < BL; ++bl) bq[h][bl] = lds16(pbase[bl] + ((h >> 1) * p.PWd + (h & 1)) * (KCS * 2) + 32 * kk);
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t so2 = kk + 1 < KSTEPS ? so + (kk + 1) * kstep : so_next; // the next step's fragments
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
#pragma unroll
                for (int bl = 0; bl < BL; ++bl) {
                    union { u32x4 u; bf16x8 v; } af, bf;
                    af.u = wr[t];
                    bf.u = bq[shift(t)][bl];
                    acc[cls(t)][bl] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf.v, af.v, acc[cls(t)][bl], 0, 0, 0);
                }
                wr[t] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, wlane, p.wofs[t] + so2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        wave_sync();
    }
    // ---- the sums of the KS waves, the two classes of a row of dX at a time, as in the kernel above
    constexpr int G = 2 * BL * 4, GK = G / KS;
    static_assert(G % KS == 0, "");
    const uint32_t out = lds0 + red2_bytes(BL, KS); // [channel][pixel][b], bfloat16
    const rsrc_t rs_out = make_rsrc(p.out, (uint32_t)p.N * p.M * p.Hout * p.Wout * 2u);
    __syncthreads(); // (all staging buffers are dead)
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int g = 0; g < G; ++g) { // g = 2 * (4 * block + group of four pixels) + b
            const int dst = g / GK;
            const f32x16 &c = acc[2 * a + (g & 1)][g / 8];
            const int jq = g / 2 % 4;
            if (dst != ks)
                *(lds_f32x4_ptr)(uintptr_t)(lds0 + (uint32_t)(((dst * (KS - 1) + (ks < dst ? ks : ks - 1)) * GK + g % GK) * 1024) + lane * 16) =
                    f32x4{c[4 * jq], c[4 * jq + 1], c[4 * jq + 2], c[4 * jq + 3]};
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g / GK != ks) continue;
            const f32x16 &c = acc[2 * a + (g & 1)][g / 8];
            const int jq = g / 2 % 4;
            f32x4 sum;
#pragma unroll
            for (int src = 0; src < KS; ++src) {
                f32x4 t = f32x4{c[4 * jq], c[4 * jq + 1], c[4 * jq + 2], c[4 * jq + 3]};
                if (src != ks) t = *(lds_f32x4_ptr)(uintptr_t)(lds0 + (uint32_t)(((ks * (KS - 1) + (src < ks ? src : src - 1)) * GK + g % GK) * 1024) + lane * 16);
                if (src == 0) sum = t;
                else sum += t;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *(lds_u16_ptr)(uintptr_t)(out + (uint32_t)(l32 * kPairRow(BL) + (g / 8 * 32 + 8 * jq + 4 * half + e) * 4 + (g & 1) * 2)) = f32_to_bf16(sum[e]);
        }
        __syncthreads();
        // a lane per pixel of dY: its pair of dX
        const int seg = threadIdx.x % PT, f = px0 + seg;
        const int gi = fdiv(f, p.m_ppi), px = f - gi * ppi, i = fdiv(px, p.m_wc), j = px - i * p.Wc, n = n0 + gi, h = 2 * i + a;
        const bool ok = (n < p.N) & (h < p.Hout);
        const uint32_t base = ((uint32_t)(n * p.M + m0) * p.Hout + h) * p.Wout + 2 * j, step = (uint32_t)p.Hout * p.Wout;
        constexpr int RPI = 64 * KS / PT; // rows at a time
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int row = it * RPI + threadIdx.x / PT;
            const uint32_t pair = *(lds_u32_ptr)(uintptr_t)(out + row * kPairRow(BL) + seg * 4);
            const uint32_t off = ok && m0 + row < p.M ? (base + row * step) * 2u : kNoLoad;
            if (p.Wout % 2 == 0) {
                __builtin_amdgcn_raw_buffer_store_b32(pair, rs_out, off, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)pair, rs_out, off, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(pair >> 16), rs_out, 2 * j + 1 < p.Wout ? off + 2 : kNoLoad, 0, 0);
            }
        }
    }
}

template <int MI, int KC, int ITEMS, int GW, int KS> hipError_t launch_fixed(const GatherParams &p, hipStream_t st)
{
    auto kern = conv_wave_kernel<MI, KC, ITEMS, GW, KS>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    GatherParams q = p;
    const dim3 grid = share_grid(q, dim3((unsigned)((p.tiles_per_img * p.mtiles + 7) / 8 * 8)), 64 * KS);
    hipLaunchKernelGGL(kern, grid, dim3(64 * KS), p.lds_bytes, st, q);
    return hipGetLastError();
}
template <int MI, int KC, int ITEMS, int KS> hipError_t launch_shape(const GatherParams &p, hipStream_t st)
{
    return p.gw == 8 ? launch_fixed<MI, KC, ITEMS, 8, KS>(p, st) : launch_fixed<MI, KC, ITEMS, 7, KS>(p, st);
}

template <int BL, int KC, int GW, int KS> hipError_t launch_dx2_fixed(const GatherParams &p, hipStream_t st)
{
    auto kern = conv_wave_dx2_kernel<BL, KC, GW, KS>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    GatherParams q = p;
    const dim3 grid = share_grid(q, dim3((unsigned)((p.tiles_per_img * p.mtiles + 7) / 8 * 8)), 64 * KS);
    hipLaunchKernelGGL(kern, grid, dim3(64 * KS), p.lds_bytes, st, q);
    return hipGetLastError();
}
template <int BL, int KC, int KS> hipError_t launch_dx2_shape(const GatherParams &p, hipStream_t st)
{
    return p.gw == 8 ? launch_dx2_fixed<BL, KC, 8, KS>(p, st) : launch_dx2_fixed<BL, KC, 7, KS>(p, st);
}

struct Shape { int mi, kc, items, ks; hipError_t (*launch)(const GatherParams &, hipStream_t); };
const Shape kShapes[] = {
    {2, 32, 1, 4, launch_shape<2, 32, 1, 4>}, {2, 16, 1, 4, launch_shape<2, 16, 1, 4>}, {2, 16, 2, 4, launch_shape<2, 16, 2, 4>},
    {1, 32, 1, 4, launch_shape<1, 32, 1, 4>}, {1, 16, 1, 4, launch_shape<1, 16, 1, 4>}, {1, 16, 2, 4, launch_shape<1, 16, 2, 4>},
    {2, 32, 1, 8, launch_shape<2, 32, 1, 8>}, {2, 16, 1, 8, launch_shape<2, 16, 1, 8>}, {2, 16, 2, 8, launch_shape<2, 16, 2, 8>},
    {1, 32, 1, 8, launch_shape<1, 32, 1, 8>}, {1, 16, 1, 8, launch_shape<1, 16, 1, 8>}, {1, 16, 2, 8, launch_shape<1, 16, 2, 8>},
};

struct Dx2Shape { int bl, kc, ks; hipError_t (*launch)(const GatherParams &, hipStream_t); };
const Dx2Shape kDx2Shapes[] = {
    {2, 32, 4, launch_dx2_shape<2, 32, 4>}, {2, 16, 4, launch_dx2_shape<2, 16, 4>}, {1, 32, 4, launch_dx2_shape<1, 32, 4>}, {1, 16, 4, launch_dx2_shape<1, 16, 4>},
    {2, 32, 8, launch_dx2_shape<2, 32, 8>}, {2, 16, 8, launch_dx2_shape<2, 16, 8>}, {1, 32, 8, launch_dx2_shape<1, 32, 8>}, {1, 16, 8, launch_dx2_shape<1, 16, 8>},
};

// Rows and images that a tile of pt pixels can reach: it starts at a multiple of pt pixels, counted over all images.  tall: rows of the
// input that an output row meets.  False where the kernels' divisions by multiplication would not be exact.
bool span_of_tile(GatherParams &p, int pt, int tall)
{
    const int ppi = p.Hc * p.Wc;
    const long tiles = ((long)p.N * ppi + pt - 1) / pt;
    if (tiles > 1 << 24) return false;
    const WaveRows r = wave_rows(p.Hin, p.Hc, p.Wc, p.is, tall, pt);
    p.VH = r.VH; p.PH = r.PH; p.IR = r.IR;
    p.tiles_per_img = (int)tiles;
    p.m_wc = magic_of(p.Wc); p.m_ppi = magic_of(ppi); p.m_ph = magic_of(p.Hin);
    p.gw = p.Win % 2 ? 7 : 8;
    p.GX = (p.Win + p.gw - 1) / p.gw;
    p.m_gx = magic_of(p.GX);
    return divides_exactly(ppi + pt, ppi) && divides_exactly(ppi, p.Wc) && divides_exactly(p.Hin + p.IR, p.Hin);
}

} // namespace

// Fills the tiling of a nine-tap launch over whole output planes; false when no shape takes it.  *cost: clock cycles, roughly.
bool shape_wave(GatherParams &p, int *variant, double *cost_out)
{
    if (p.ntaps != TAPS || p.os != 1 || p.Hc != p.Hout || p.Wc != p.Wout) return false;
    GatherParams b = p;
    b.dhmin = b.dwmin = 1 << 30;
    int dhmax = -(1 << 30), dwmax = -(1 << 30);
    for (int t = 0; t < TAPS; ++t) {
        if (p.wtap[t] != t) return false;
        b.dhmin = min(b.dhmin, p.dh[t]); dhmax = max(dhmax, p.dh[t]);
        b.dwmin = min(b.dwmin, p.dw[t]); dwmax = max(dwmax, p.dw[t]);
    }
    const int ppi = p.Hc * p.Wc, tall = dhmax - b.dhmin + 1;
    b.PWd = (p.Wc - 1) * p.is + (dwmax - b.dwmin) + 1;
    b.ksplit = 1; b.T = 1; b.part = nullptr; b.gpw = 1; b.IPT = 1;
    if (!span_of_tile(b, PT, tall)) return false;
    const long tiles = b.tiles_per_img;
    b.store_px = ppi % 8 == 0 ? 8 : ppi % 4 == 0 ? 4 : ppi % 2 == 0 ? 2 : 1;
    int force = -1;
#ifdef CAC_TUNING
    if (const char *f = getenv("CAC_WAVE_SHAPE")) force = atoi(f);
#endif
    GatherParams best{};
    double best_cost = 1e300;
    for (int v = 0; v < (int)(sizeof(kShapes) / sizeof(kShapes[0])); ++v) {
        const Shape &sh = kShapes[v];
        if (force >= 0 && v != force) continue;
        GatherParams q = b;
        const int items = b.IR * b.GX * (sh.kc / 8), kcs = sh.kc + 8;
        if (items > 64 * sh.items || (sh.items == 2 && items <= 64)) continue;
        q.patch_px = q.PH * q.PWd;
        q.buf_bytes = (q.patch_px * kcs * 2 + 15) / 16 * 16;
        q.lds_bytes = max(sh.ks * (q.buf_bytes + 64 * 16), red_bytes(sh.mi, sh.ks) + 32 * sh.mi * kOutRow);
        if (q.lds_bytes > 160 * 1024) continue;
        q.KCp = (p.KCin + sh.kc - 1) / sh.kc * sh.kc;
        q.nkb = q.KCp / sh.kc;
        q.kbs = (q.nkb + sh.ks - 1) / sh.ks; // (stages of the busiest wave)
        q.mtiles = (p.M + 32 * sh.mi - 1) / (32 * sh.mi);
        for (int t = 0; t < TAPS; ++t) {
            q.wofs[t] = (uint32_t)t * (q.KCp / 16) * (q.Mp / 32) * kFrag;
            q.toff[t] = (uint32_t)((p.dh[t] - q.dhmin) * q.PWd + (p.dw[t] - q.dwmin)) * kcs * 2u;
        }
        const int resident = min(8 / sh.ks, 160 * 1024 / q.lds_bytes); // workgroups of a compute unit
        const long wgs = tiles * q.mtiles, rounds = (wgs + 256L * resident - 1) / (256L * resident);
        const double busy = (double)min((long)resident * sh.ks, ((wgs + 255) / 256) * sh.ks) / 4; // waves of a SIMD
        const double step = max(32.0 * NI * sh.mi * max(1.0, busy), 150.0);
        const double cost = rounds * (q.kbs * (TAPS * (sh.kc / 16) * step + 800.0) + 5000.0 + (sh.ks == 8 ? 800.0 : 0.0));
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

// ... of the 3 x 3 stride-2 data gradient with padding 1.  p: N, M (= C_in), Mp, KCin (= C_out), Hin, Win (of dY), Hout, Wout (of dX) are filled in.
bool shape_wave_dx2(const Geom &g, GatherParams &p, int *variant, double *cost_out)
{
    if (g.R != 3 || g.S != 3 || g.sh != 2 || g.sw != 2 || g.ph != 1 || g.pw != 1) return false;
    GatherParams b = p;
    b.Hc = g.P; b.Wc = g.Q;
    b.dhmin = b.dwmin = 0;
    b.PWd = g.Q + 1;
    b.os = 2; b.is = 1; b.ntaps = b.ntaps_total = TAPS;
    b.ksplit = 1; b.T = 1; b.part = nullptr; b.gpw = 1; b.IPT = 1;
    int force = -1;
#ifdef CAC_TUNING
    if (const char *f = getenv("CAC_WAVE_DX2_SHAPE")) force = atoi(f);
#endif
    GatherParams best{};
    double best_cost = 1e300;
    for (int v = 0; v < (int)(sizeof(kDx2Shapes) / sizeof(kDx2Shapes[0])); ++v) {
        const Dx2Shape &sh = kDx2Shapes[v];
        if (force >= 0 && v != force) continue;
        GatherParams q = b;
        if (!span_of_tile(q, 32 * sh.bl, 2) || q.IR * q.GX * (sh.kc / 8) > 64) continue;
        const int kcs = sh.kc + 8;
        q.patch_px = q.PH * q.PWd;
        q.buf_bytes = (q.patch_px * kcs * 2 + 15) / 16 * 16;
        q.lds_bytes = max(sh.ks * (q.buf_bytes + 64 * 16), red2_bytes(sh.bl, sh.ks) + 32 * kPairRow(sh.bl));
        if (q.lds_bytes > 160 * 1024) continue;
        q.KCp = (p.KCin + sh.kc - 1) / sh.kc * sh.kc;
        q.nkb = q.KCp / sh.kc;
        q.kbs = (q.nkb + sh.ks - 1) / sh.ks;
        q.mtiles = (p.M + 31) / 32;
        for (int t = 0; t < TAPS; ++t) q.wofs[t] = (uint32_t)t * (q.KCp / 16) * (q.Mp / 32) * kFrag;
        const int resident = min(8 / sh.ks, 160 * 1024 / q.lds_bytes);
        const long wgs = (long)q.tiles_per_img * q.mtiles, rounds = (wgs + 256L * resident - 1) / (256L * resident);
        const double busy = (double)min((long)resident * sh.ks, ((wgs + 255) / 256) * sh.ks) / 4;
        const double step = max(TAPS * 32.0 * sh.bl * max(1.0, busy), 800.0); // of 16 channels
        const double cost = rounds * (q.kbs * ((sh.kc / 16) * step + 800.0) + 6500.0 + (sh.ks == 8 ? 800.0 : 0.0));
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

hipError_t launch_wave_dx2(const GatherParams &p, int variant, hipStream_t st) { return kDx2Shapes[variant].launch(p, st); }

int describe_wave_dx2(const GatherParams &p, int variant, char *buf, size_t len)
{
    const Dx2Shape &v = kDx2Shapes[variant];
    return snprintf(buf, len, "tile=32ch x 4 x %dpx by waves (four parity classes, %d share the channels, stages of %d) taps=9 rows/tile=%d grid=%dx%dx1 lds=%dB",
                    32 * v.bl, v.ks, v.kc, p.IR, p.tiles_per_img, p.mtiles, p.lds_bytes);
}

hipError_t launch_wave(const GatherParams &p, int variant, hipStream_t st) { return kShapes[variant].launch(p, st); }

int describe_wave(const GatherParams &p, int variant, char *buf, size_t len)
{
    const Shape &v = kShapes[variant];
    return snprintf(buf, len, "tile=%dch x %dpx by waves (%d share the channels, stages of %d) taps=%d rows/tile=%d grid=%dx%dx1 lds=%dB, input read in place",
                    32 * v.mi, PT, v.ks, v.kc, p.ntaps, p.IR, p.tiles_per_img, p.mtiles, p.lds_bytes);
}

} // namespace cac
