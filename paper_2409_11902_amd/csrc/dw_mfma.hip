// Weight gradient from the compressed activation as an MFMA implicit GEMM
// (bfloat16 operands, float accumulation), gfx950.
//
//   dW[o,c,r,s] = sum_{n,p,q} dY[n,o,p,q] * xhat[n,c,p*SG+r-PAD,q*SG+s-PAD],
//   xhat[n,c,h,w] = Z[n,c,h/kh,w/kw]        (weight-gradient formula of the
//                                             compression figure; inflation by
//                                             replication)
//
// GEMM view: M = output channels o, N = (input channel c, filter tap), K = pixels.
// A workgroup owns a (32*MI*WM) x (32*NI*WN) x all-taps tile and a slice of the
// pixels.  It has WM*WN*KS MFMA waves -- each holding MI x NI x taps accumulator
// blocks of 32x32; the KS waves that share a block split the rows of every chunk
// and add up through LDS at the end -- and as many copy waves, which bring the
// operands from global memory into LDS (one MFMA and one copy wave per SIMD).
//
// The pixel sum is re-indexed by the xhat column instead of the output column:
// with s - PAD = SG*a_s + b_s (0 <= b_s < SG),
//   dW[o,c,r,s] = sum_{n,p,j} dY[n,o,p,j-a_s] * xhat[n,c,p*SG+r-PAD, SG*j+b_s]
// so the xhat operand is always an ALIGNED block of 8 columns of "phase" b_s of
// an xhat row (phase b holds columns b, b+SG, ...), and only the dY operand is
// shifted (by a_s = -1, 0 or +1 columns).  One shifted dY fragment serves all
// filter rows and input-channel blocks; it is made in registers with v_perm from
// a sliding window over the dY row.  Zero padding needs no halo: columns outside
// the image simply do not occur, pixels outside the row are zero in the window.
// A 32x32x16 MFMA consumes two such blocks of 8, one in lanes 0-31 and one in
// lanes 32-63 (rows rho and rho+1 of the staged chunk).
//
// Staging per chunk (NBI images x PR output rows), double buffered in LDS:
//   rows [LR]                      per row: LDS offsets of its dY row and of the
//                                  xhat rows feeding each filter row
//   sDY  [tile_o][LR rows][Qpad]   dY, rows padded with zeros to a multiple of 8
//   sX   [tile_c][slots][phase][Qpad]  the needed rows of Z, expanded along the
//                                  row to full input width, zeros past W
// plus one shared all-zero row.  The inflated activation exists only here:
// expanded horizontally when written to LDS, expanded vertically by mapping an
// input row h to the slot of Z row h/kh.

#include <mutex>
#include <type_traits>

#include "common.h"
#include "dw_mfma.h"
#include "dw_reduce.h"

namespace cac {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

__device__ __forceinline__ uint32_t fdiv(uint32_t x, uint32_t magic) { return magic ? __umulhi(x, magic) : x; }

__device__ __forceinline__ uint32_t pack16(uint32_t lo, uint32_t hi) { return (lo & 0xffffu) | (hi << 16); }

// Result: low half = half `ha` of a, high half = half `hb` of b.
template <int ha, int hb> __device__ __forceinline__ uint32_t halves(uint32_t a, uint32_t b)
{
    constexpr uint32_t sel = (2 * ha) | ((2 * ha + 1) << 8) | ((4 + 2 * hb) << 16) | ((5 + 2 * hb) << 24);
    return __builtin_amdgcn_perm(b, a, sel);
}

// 16 bytes of LDS at an absolute LDS byte address (saves the compiler adding the
// base of the dynamic LDS block, unknown until link time, to every access).
typedef __attribute__((address_space(3))) const u32x4 *lds_u32x4_ptr;
__device__ __forceinline__ u32x4 lds16(uint32_t addr) { return *(lds_u32x4_ptr)(uintptr_t)addr; }

// 16-byte items of dY and of Z a thread moves per chunk, at most (every chunk issues so many loads, wanted or not).
// Uncompressed records of 3 x 3 stride-2 layers (pooling tiles of one column) hold many Z items to every dY item: with the
// split of the others a chunk is one output row on wide maps, half of a row pair left empty; under stride 1 they hold two rows more
// than a chunk has of dY.  WIDEZ 1 and 2 are the other splits:
// longer chunks, but a workgroup waits for more before its first; dw_mfma_plan draws the lines.
constexpr int max_dy(int widez) { return 8 >> widez; }
constexpr int max_z(int widez) { return 4 << widez; }

// A window of one xhat row held in registers: the last dword of the block left
// of the current position and NB blocks starting at it.
template <int NB> struct Window {
    uint32_t prev3;
    u32x4 blk[NB];
};

// Element `e` (relative to the first element of blk[0]; -2 <= e < 8*NB): its register.
template <int NB, int e> __device__ __forceinline__ uint32_t win_reg(const Window<NB> &w)
{
    static_assert(e >= -2 && e < 8 * NB, "window too small");
    if constexpr (e < 0)
        return w.prev3;
    else
        return w.blk[e / 8][(e % 8) / 2];
}
template <int e> constexpr int win_half() { return ((e % 2) + 2) % 2; }

// B fragment for filter column s: pixel j of the segment needs element
// SG*j + s - PAD of the window.
template <int NB, int SG, int PAD, int s> __device__ __forceinline__ bf16x8 make_frag(const Window<NB> &w)
{
    union { u32x4 u; bf16x8 v; } f;
#define CAC_FRAG_DWORD(i)                                                                            \
    {                                                                                                \
        constexpr int e0 = SG * (2 * i) + s - PAD, e1 = SG * (2 * i + 1) + s - PAD;                  \
        if constexpr (e0 >= 0 && e0 % 2 == 0 && e1 == e0 + 1)                                        \
            f.u[i] = win_reg<NB, e0>(w); /* both halves of one dword, in place */                    \
        else                                                                                         \
            f.u[i] = halves<win_half<e0>(), win_half<e1>()>(win_reg<NB, e0>(w), win_reg<NB, e1>(w)); \
    }
    CAC_FRAG_DWORD(0) CAC_FRAG_DWORD(1) CAC_FRAG_DWORD(2) CAC_FRAG_DWORD(3)
#undef CAC_FRAG_DWORD
    return f.v;
}

// Global reads go through buffer loads: a lane whose byte offset lies at or beyond
// the tensor's size gets zeros back without touching memory and without a branch,
// so every load of a chunk can be in flight at once (tensors on this path are
// smaller than 2 GiB; offsets from 2^31 on mean "no load").
// Items are read with one 16-byte load each from the dword-aligned address at or below
// their first element (rows of odd length start on odd elements).
// The 8 elements themselves, of items `d` at elements e, e + step, ...  After an odd start everything moves down by one
// element and the last one comes from the first dword of the next item of the
// same row, which the next lane holds (the copy maps consecutive items of a row
// to consecutive lanes; the last item of a row never needs it: a row of odd
// length ends before its 8th element; `multi`: a row has several).  Then ANDed with `mask`: zero from the
// row's end on, what follows belongs to another row.
template <int N> __device__ __forceinline__ void fix8(u32x4 (&v)[N], const u32x4 (&d)[N], uint32_t e, uint32_t step, const u32x4 &mask, bool multi)
{
    uint32_t next0[N];
#pragma unroll
    for (int i = 0; i < N; ++i) next0[i] = d[i][0];
    if (multi) {
#pragma unroll
        for (int i = 0; i < N; ++i) next0[i] = __shfl_down(d[i][0], 1, 64);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t sh = ((e + i * step) & 1u) * 16u;
        v[i] = u32x4{__builtin_amdgcn_alignbit(d[i][1], d[i][0], sh), __builtin_amdgcn_alignbit(d[i][2], d[i][1], sh),
                     __builtin_amdgcn_alignbit(d[i][3], d[i][2], sh), __builtin_amdgcn_alignbit(next0[i], d[i][3], sh)} & mask;
    }
}
// Dword j of the mask keeps the elements 2j, 2j+1 that lie below `left`.
__device__ __forceinline__ u32x4 mask8(int left)
{
    u32x4 m;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int l2 = left - 2 * j;
        m[j] = l2 >= 2 ? 0xffffffffu : (l2 == 1 ? 0xffffu : 0u);
    }
    return m;
}

// FL: log2 of the columns of one phase that a pooled value covers; -1: half a column, an uncompressed record under stride
// 2.  Built in: with all forms of the expansion in one kernel the copy waves of two phases spilled 158 registers (WIDEZ: 233) to
// scratch, more traffic than the operands -- 128 -> 256 at 28 x 28, batch 128, uncompressed 61 -> 42 us; 150 random layers, tiles of 1, 2
// and 4, 0.72 of the time, none slower --, and those of one phase went through 70 KB of code, more than the instruction cache
// holds (250 random 3 x 3 stride-1 layers, uncompressed: 0.92 of the time, none slower).
// SC: the number of 8-pixel segments per output row when it is known at compile
// time (0: read from the plan).  With SC the walk along a row is unrolled and the
// segment offsets become immediates of the LDS reads.
template <int R, int S, int SG, int PAD, int MI, int NI, int WM, int WN, int KS, int SC, bool DYL, int WIDEZ, int FL>
__global__ void __launch_bounds__(128 * WM * WN * KS) dw_mfma_kernel(DwMfmaParams p, RepackParams rep)
{
    constexpr int kMaxDy = max_dy(WIDEZ), kMaxZ = max_z(WIDEZ);
    constexpr int T = R * S;
    constexpr int NT = 64 * WM * WN * KS; // threads of each kind: MFMA waves, then as many copy waves
    constexpr int TILE_O = 32 * MI * WM, TILE_C = 32 * NI * WN;
    // floor division / remainder of (s - PAD) by SG for every filter column
    constexpr auto a_of = [](int s) { int d = s - PAD; return d >= 0 ? d / SG : -((-d + SG - 1) / SG); };
    constexpr auto b_of = [](int s) { int d = s - PAD; return d - SG * (d >= 0 ? d / SG : -((-d + SG - 1) / SG)); };
    constexpr int NPH = (S == 1) ? 1 : SG; // xhat column phases in use
    static_assert(S <= 3 && SG <= 2 && a_of(0) >= -1 && a_of(S - 1) <= 1, "unsupported filter geometry");

    extern __shared__ __align__(16) unsigned char smem[];
    // [zero row][buffer 0: rows, sDY, sX][buffer 1: rows, sDY, sX]; offsets below are in
    // bf16 elements from the start of LDS, so offset 0 is the zero row
    bf16_t *sW = (bf16_t *)smem;
    // Every cache line of the arguments is asked for here, in one go (each would be a round trip of its own where it is first needed).
    asm volatile("" ::"s"(p.own_wgs), "s"(p.NBI), "s"(p.LDY), "s"(p.nchunks));
    const uint32_t rows_elems = p.LRpad * 8;                   // one 16-byte entry per row
    const uint32_t buf_elems = rows_elems + TILE_O * p.dy_ostride + TILE_C * p.x_cstride;
    const uint32_t slot_w = NPH * p.PW;                        // one xhat row: all phases
    const uint32_t base0 = slot_w, base1 = base0 + buf_elems;  // the buffers follow the zero row

    if constexpr (NT == 256) {
        // Past the kernel's own workgroups: what the data gradient of the same layer needs laid out ahead of it, on compute units
        // that a small layer leaves idle (launch_dw_mfma).
        if (__builtin_expect(blockIdx.x >= p.own_wgs, 0)) {
            const int sub = threadIdx.x >> 8;
            repack_body(rep, 2 * (blockIdx.x - p.own_wgs) + sub, (bf16_t *)smem + sub * kRepackElems, threadIdx.x & 255);
            return;
        }
    }
    // Workgroups are dealt round-robin to the 8 XCDs; renumber them so that each
    // XCD works on consecutive (slice, o-tile, c-tile) triples and re-reads of dY
    // and Z hit its own L2.
    const int per_xcd = p.own_wgs >> 3;
    const int v = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (v >= p.total_wg) return;
    const int ntiles = p.tiles_o * p.tiles_c;
    const int slice = v / ntiles, tile = v - slice * ntiles;
    const int ot = tile / p.tiles_c, ct = tile - ot * p.tiles_c;
    const int o0 = ot * TILE_O, c0 = ct * TILE_C;

    // What is read without ever being staged must start as zero: the shared zero row and,
    // in both buffers, the xhat part (every channel ends with an all-zero slot).  The row
    // table and the dY part are rewritten in full for every chunk.
    auto zero_fill = [&]() {
        const uint32_t x_elems = TILE_C * p.x_cstride, x_off = rows_elems + TILE_O * p.dy_ostride;
        u32x4 *l = (u32x4 *)smem;
        for (uint32_t i = threadIdx.x; i < slot_w / 8; i += 2 * NT) l[i] = u32x4{0, 0, 0, 0};
        for (uint32_t i = threadIdx.x; i < x_elems / 8; i += 2 * NT) {
            l[(base0 + x_off) / 8 + i] = u32x4{0, 0, 0, 0};
            l[(base1 + x_off) / 8 + i] = u32x4{0, 0, 0, 0};
        }
    };

    const int ci_begin = slice * p.chunks_per_slice;
    const int ci_end = min(ci_begin + p.chunks_per_slice, p.nchunks);

    // the role of a wave is uniform over the wave: tell the compiler so
    const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave_id >= NT / 64) {
        // =========================== copy waves ===========================================
        // They keep two chunks of global loads in flight and fill the LDS buffer the
        // MFMA waves are not reading; the only hand-over is one barrier per chunk.  Where a chunk has less than 3500 cycles of
        // MFMAs these waves bound it, not by waiting for memory (100 cycles) but by what they issue: 1100-1900 cycles for dY, 1000-1500
        // for Z, 800 for the loads, which the address unit takes at 64 bytes a cycle.
        const int tid = threadIdx.x - NT;
        // dY: LDY lanes share one output channel's rows; item j = (row rho, segment sg)
        const uint32_t dyj = tid & (p.LDY - 1), dyo = tid >> p.ldy_log2;
        const uint32_t dy_rho = fdiv(dyj, p.m_segs), dy_sg = dyj - dy_rho * p.SEGS;
        const uint32_t dy_ni = fdiv(dy_rho, p.m_pr), dy_pr = dy_rho - dy_ni * p.PR;
        const bool dy_write = dyj < (uint32_t)p.rowitems;         // lanes past the row's items idle
        const bool dy_real = dy_write && dy_rho < (uint32_t)p.LR; // the spare row stays zero
        u32x4 dy_mask, z_mask, rag[2][2]; // (filled after the first loads are on their way)
        const uint32_t dy_rel = ((dy_ni * p.K + dyo) * p.P + dy_pr) * p.Q + dy_sg * 8;
        const uint32_t dy_opp = (uint32_t)NT >> p.ldy_log2;       // output channels per pass
        const uint32_t dy_gstep = dy_opp * p.P * p.Q;
        const uint32_t dy_lds = rows_elems + dyo * p.dy_ostride + dyj * 8;
        const uint32_t dy_lstep = dy_opp * p.dy_ostride;
        // Z: LPC lanes share one input channel; item j = (image ni, slot sl, vector zv of 8 pooled values)
        const uint32_t zj = tid & (p.LPC - 1), zc = tid >> p.lpc_log2;
        const uint32_t z_row = fdiv(zj, p.m_zv), z_zv = zj - z_row * p.ZV;
        const uint32_t z_ni = fdiv(z_row, p.m_nz), z_sl = z_row - z_ni * p.NZ;
        const bool z_write = zj < (uint32_t)p.citems;
        const uint32_t z_rel = ((z_ni * p.C + zc) * p.Hp + z_sl) * p.Wp + z_zv * 8;
        const uint32_t z_cpp = (uint32_t)NT >> p.lpc_log2;        // input channels per pass
        const uint32_t z_gstep = z_cpp * p.Hp * p.Wp;
        const uint32_t z_lds = rows_elems + TILE_O * p.dy_ostride + zc * p.x_cstride + z_row * slot_w;
        const uint32_t z_lstep = z_cpp * p.x_cstride;
        const bool dy_odd = p.Q & 1, z_odd = p.Wp & 1;
        const bool ragged = (p.W & ((1 << p.kw_log2) - 1)) != 0; // the last pooling tile reaches past W
        const rsrc_t rs_dy = make_rsrc(p.dY, (uint32_t)p.N * p.K * p.P * p.Q * 2u);
        const rsrc_t rs_z = make_rsrc(p.Z, (uint32_t)p.N * p.C * p.Hp * p.Wp * 2u);
        // Output channels past K and input channels past C of an edge tile are read like any
        // other (from whatever follows in the tensor, zeros past its end): they only reach
        // accumulators that are never written out.

        // What depends on the chunk is uniform over the workgroup: the first image and output
        // row, the first Z row kept, and the element offsets of the tile's first dY / Z element.
        struct Src { uint32_t dy, z; int zbase, n0, p0; };
        auto src_of = [&](int ci) {
            Src s;
            const int ig = fdiv(ci, p.m_rb), rb = ci - ig * p.RB;
            s.n0 = ig * p.NBI;
            s.p0 = rb * p.PR;
            s.zbase = max(0, (s.p0 * SG - PAD) >> p.kh_log2);
            s.dy = ((uint32_t)(s.n0 * p.K + o0) * p.P + s.p0) * p.Q;
            s.z = ((uint32_t)(s.n0 * p.C + c0) * p.Hp + s.zbase) * p.Wp;
            return s;
        };
        // Element offset of this lane's item within the chunk, or far outside the tensor
        // (2^30 elements: the byte offset stays in [2^31, 2^32) after every addition below)
        // for a lane without an item.
        constexpr uint32_t kNoElem = 0x40000000u;
        const uint32_t dy_lane = dy_real ? dy_rel : kNoElem, z_lane = z_write ? z_rel : kNoElem;
        const uint32_t dy_istep = dy_gstep, z_istep = z_gstep;
        // ---- global -> registers for one chunk: one add per item, no branch
        // `live` false (uniform): the chunk does not exist; the loads are issued all the same,
        // past the tensors, so that the number of loads in flight is the same on every path and
        // a wait for the older chunk never has to include the younger one.
        auto fetch = [&](int ci, bool live, u32x4 (&rdy)[kMaxDy], u32x4 (&rz)[kMaxZ]) {
            const Src s = src_of(ci);
            // rows past P and images past N of an edge chunk must read as zeros: their pixels
            // meet real xhat rows in the shifted windows of their neighbours
            const bool dy_in = live && s.n0 + (int)dy_ni < p.N && s.p0 + (int)dy_pr < p.P;
            const uint32_t e_dy = dy_in ? s.dy + dy_lane : kNoElem;
            const uint32_t e_z = live ? s.z + z_lane : kNoElem; // rows past Hp are never looked at
            if constexpr (!DYL) {
#pragma unroll
                for (int i = 0; i < kMaxDy; ++i) {
                    // items past the last pass: offset 2^30 elements as well (uniform select)
                    const uint32_t e = e_dy + (i < p.dy_passes ? i * dy_istep : kNoElem);
                    rdy[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_dy, (e & ~1u) * 2u, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < kMaxZ; ++i) {
                const uint32_t e = e_z + (i < p.z_passes ? i * z_istep : kNoElem);
                rz[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_z, (e & ~1u) * 2u, 0, 0);
            }
        };
        const int cw = __builtin_amdgcn_readfirstlane(tid >> 6); // index among the copy waves
        // DYL: dY goes from global memory straight into the LDS buffer (no registers, no LDS
        // store instructions).  A load of this kind writes the 64 lanes' 16 bytes side by side
        // from a uniform LDS address on, which is this kernel's dY layout when a wave's 64
        // lanes are the 64 items of one output channel and no item needs a mask (the plan sets
        // dy_direct then); lanes without a row, and chunks that do not exist, load zeros.
        auto load_dy = [&](int ci, bool live, uint32_t base) {
            const Src s = src_of(ci);
            const bool dy_in = live && s.n0 + (int)dy_ni < p.N && s.p0 + (int)dy_pr < p.P;
            const uint32_t e_dy = dy_in ? s.dy + dy_lane : kNoElem;
            __attribute__((address_space(3))) unsigned char *l3 = (__attribute__((address_space(3))) unsigned char *)smem;
#pragma unroll
            for (int i = 0; i < kMaxDy; ++i) {
                const uint32_t off = __builtin_amdgcn_readfirstlane((base + rows_elems + (cw + i * dy_opp) * p.dy_ostride) * 2u);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_dy, (__attribute__((address_space(3))) void *)(l3 + off), 16,
                                                         (e_dy + i * dy_istep) * 2u, 0, 0, 0);
            }
        };
        // DYL: everything but the Z loads of the youngest fetch has arrived, this chunk's dY too
        auto dy_landed = [&]() { __builtin_amdgcn_s_waitcnt((kMaxZ & 0xF) | ((kMaxZ >> 4) << 14) | 0x0F70); };
        // ---- registers -> LDS buffer at element offset `base` (with the horizontal inflation)
        auto stage = [&](int ci, uint32_t base, const u32x4 (&rdy)[kMaxDy], const u32x4 (&rz)[kMaxZ]) {
            // Everything but the kMaxDy + kMaxZ loads of the younger chunk has arrived.  Said
            // explicitly: items past the last pass are loaded but never looked at, and the
            // compiler, seeing loads nobody waited for, would otherwise drain the whole queue
            // before reusing their registers.  (s_waitcnt operand: vmcnt in bits 3:0 and 15:14,
            // the other counters left at their maximum.)
            constexpr int kYounger = kMaxDy + kMaxZ;
            __builtin_amdgcn_s_waitcnt((kYounger & 0xF) | ((kYounger >> 4) << 14) | 0x0F70);
            const Src s = src_of(ci);
            // row table: entry rho = {dY row offset, xhat row offset per filter row (the zero
            // slot for rows outside the image)}, in elements from the lane's channel base.  Chunks of whole images
            // have the same one but for the last (400 cycles of the 3500 that a chunk takes this wave, which is behind the others by them;
            // under stride 2, where chunks of parts of an image are the rule, the question alone costs 128 -> 256 at 28 x 28, batch 128,
            // uncompressed, 43.8 against 43.4 us, and 60 random layers are even without it)
            const bool same = SG == 1 && p.RB == 1 && ci >= ci_begin + 2 && s.n0 + p.NBI <= p.N;
            if (cw == 0 && !same && tid < p.LRpad) {
                const uint32_t rho = tid;
                const uint32_t ni = fdiv(rho, p.m_pr);
                const int pp = s.p0 + (int)(rho - ni * p.PR);
                const bool row_ok = rho < (uint32_t)p.LR && pp < p.P && s.n0 + (int)ni < p.N;
                const uint32_t zero_slot = p.NBI * p.NZ * slot_w; // each channel ends with an all-zero xhat row
                u32x4 e = {rho * (uint32_t)p.Qpad, zero_slot, zero_slot, zero_slot};
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int h = pp * SG + r - PAD;
                    const bool ok = row_ok && h >= 0 && h < p.H;
                    e[1 + r] = ok ? ((int)ni * p.NZ + (h >> p.kh_log2) - s.zbase) * slot_w : zero_slot;
                }
                *(u32x4 *)(sW + base + rho * 8) = e;
            }
            // dY: fix-ups for all items first (they exchange data between lanes), then one
            // predicated run of stores
            u32x4 val[kMaxDy];
            if constexpr (DYL) {
            } else if (dy_odd) {
                fix8(val, rdy, s.dy + dy_rel, dy_istep, dy_mask, p.SEGS > 1);
            } else {
#pragma unroll
                for (int i = 0; i < kMaxDy; ++i) val[i] = rdy[i] & dy_mask;
            }
            if (!DYL && dy_write) {
                bf16_t *d = sW + base + dy_lds;
#pragma unroll
                for (int i = 0; i < kMaxDy; ++i)
                    if (i < p.dy_passes) *(u32x4 *)(d + i * dy_lstep) = val[i];
            }
            // Z
            u32x4 zz[kMaxZ];
            if (z_odd) {
                fix8(zz, rz, s.z + z_rel, z_istep, z_mask, p.ZV > 1);
            } else {
#pragma unroll
                for (int i = 0; i < kMaxZ; ++i) zz[i] = rz[i] & z_mask;
            }
            if (z_write) {
                bf16_t *zd = sW + base + z_lds;
                // Writes 8 elements of phase ph starting at element j; in the ragged case the
                // elements whose xhat column SG*j+ph is at or beyond W are zeroed.
                auto put8 = [&](bf16_t *dst, int ph, int j, u32x4 x) {
                    if (ragged) x &= mask8((p.W - ph + SG - 1) / SG - j);
                    *(u32x4 *)(dst + ph * p.PW + j) = x;
                };
#define CAC_Z_ITEMS(...)                                                                           \
    _Pragma("unroll") for (int i = 0; i < kMaxZ; ++i) if (i < p.z_passes)                          \
    {                                                                                              \
        const u32x4 z = zz[i];                                                                     \
        bf16_t *dst = zd + i * z_lstep;                                                            \
        /* pooled value k of the item in both halves of a dword */                                 \
        auto dup = [&](int k) { return (k & 1) ? halves<1, 1>(z[k >> 1], z[k >> 1]) : halves<0, 0>(z[k >> 1], z[k >> 1]); }; \
        (void)dup;                                                                                 \
        __VA_ARGS__                                                                                \
    }
                if constexpr (FL < 0) {
                    // kw = 1, stride 2: even columns to phase 0, odd ones to phase 1
                    // (zeros past W come from the load)
                    const int j0 = z_zv * 4;
                    CAC_Z_ITEMS({
                        *(u32x2 *)(dst + j0) = u32x2{halves<0, 0>(z[0], z[1]), halves<0, 0>(z[2], z[3])};
                        if (NPH > 1) *(u32x2 *)(dst + p.PW + j0) = u32x2{halves<1, 1>(z[0], z[1]), halves<1, 1>(z[2], z[3])};
                    })
                } else if constexpr (FL == 0) {
                    const int j0 = z_zv * 8;
                    CAC_Z_ITEMS({
                        _Pragma("unroll") for (int ph = 0; ph < NPH; ++ph)
                            *(u32x4 *)(dst + ph * p.PW + j0) = ragged ? z & rag[ph][0] : z;
                    })
                } else if constexpr (FL == 1) {
                    const int j0 = z_zv * 16;
                    CAC_Z_ITEMS({
                        const u32x4 lo = {dup(0), dup(1), dup(2), dup(3)}, hi = {dup(4), dup(5), dup(6), dup(7)};
                        _Pragma("unroll") for (int ph = 0; ph < NPH; ++ph) {
                            *(u32x4 *)(dst + ph * p.PW + j0) = ragged ? lo & rag[ph][0] : lo;
                            *(u32x4 *)(dst + ph * p.PW + j0 + 8) = ragged ? hi & rag[ph][1] : hi;
                        }
                    })
                } else if constexpr (FL == 2) {
                    const int j0 = z_zv * 32;
                    CAC_Z_ITEMS({
                        _Pragma("unroll") for (int g = 0; g < 4; ++g) {
                            const u32x4 x = {dup(2 * g), dup(2 * g), dup(2 * g + 1), dup(2 * g + 1)};
                            _Pragma("unroll") for (int ph = 0; ph < NPH; ++ph) put8(dst, ph, j0 + 8 * g, x);
                        }
                    })
                } else {
                    const int j0 = z_zv * 64;
                    CAC_Z_ITEMS({
                        _Pragma("unroll") for (int g = 0; g < 8; ++g) {
                            const u32x4 x = {dup(g), dup(g), dup(g), dup(g)};
                            _Pragma("unroll") for (int ph = 0; ph < NPH; ++ph) put8(dst, ph, j0 + 8 * g, x);
                        }
                    })
                }
#undef CAC_Z_ITEMS
            }
        };

        u32x4 dyA[kMaxDy], zA[kMaxZ], dyB[kMaxDy], zB[kMaxZ];
        // Two chunks of loads are in flight.  A register set is refilled right after it has been
        // staged, in the same straight-line code, so that the compiler sees every load consumed
        // before its register is reused and never has to drain the other set's loads.
        fetch(ci_begin, true, dyA, zA); // (every workgroup has at least one chunk)
        fetch(ci_begin + 1, ci_begin + 1 < ci_end, dyB, zB);
        // what only the staging needs: the masks that cut an item at the end of its row, and,
        // for the ragged case, the two blocks an item expands to when FL <= 1
        dy_mask = mask8(p.Q - (int)dy_sg * 8);
        z_mask = mask8(p.Wp - (int)z_zv * 8);
#pragma unroll
        for (int ph = 0; ph < 2; ++ph)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                rag[ph][h] = mask8((p.W - ph + SG - 1) / SG - (int)(z_zv << (3 + max(FL, 0))) - 8 * h);
        if constexpr (DYL) load_dy(ci_begin, true, base0);
        zero_fill(); // in the shadow of the first loads
        __syncthreads();
        for (int ci = ci_begin;; ci += 2) {
            // MFMA waves are on buffer 1 (chunk ci-1); set A holds chunk ci, set B chunk ci+1
            if (DYL && ci != ci_begin) load_dy(ci, true, base0); // (buffer 0 is free since the last barrier)
            stage(ci, base0, dyA, zA);
            fetch(ci + 2, ci + 2 < ci_end, dyA, zA);
            if constexpr (DYL) dy_landed();
            __syncthreads();
            if (ci + 1 >= ci_end) break;
            // MFMA waves are on buffer 0 (chunk ci); set B holds chunk ci+1, set A chunk ci+2
            if constexpr (DYL) load_dy(ci + 1, true, base1);
            stage(ci + 1, base1, dyB, zB);
            fetch(ci + 3, ci + 3 < ci_end, dyB, zB);
            if constexpr (DYL) dy_landed();
            __syncthreads();
            if (ci + 2 >= ci_end) break;
        }
        __syncthreads(); // the MFMA waves' last chunk
        if constexpr (KS > 1) __syncthreads(); // the barrier inside the MFMA waves' cross-wave sum
        return;
    }

    // =============================== MFMA waves ===========================================
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id;
    const int wm = wave % WM, wn = (wave / WM) % WN, ks = wave / (WM * WN), half = lane >> 5, l32 = lane & 31;

    // The data gradient's filter, while the first chunk is on its way to LDS (2.7-3.3 us): a wave by itself per block of it, in
    // the part of buffer 1 that holds dY later on, which nobody clears, or past the buffers.
    if (NT == 256 && __builtin_expect(wave < p.rep_waves, 0))
        for (int b = v * p.rep_waves + wave; b < p.rep_blocks; b += p.total_wg * p.rep_waves)
            filter_repack_wave(rep.f, b, sW + p.rep_at + wave * p.rep_elems, lane);
    zero_fill();
    __syncthreads();

    f32x16 acc[MI][NI][T];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int j = 0; j < 16; ++j) acc[mi][ni][t][j] = 0.f;

    // ---- MFMA over one staged chunk --------------------------------------------------
    // Operands of one step: the window over the dY row(s) and the xhat blocks.
    struct Ops {
        Window<2> aw[MI];
        u32x4 b[R][NI][NPH];
    };
    // the MFMAs of one filter column of a step: the window supplies the shifted dY fragments
    auto mfma_cols = [&](const Ops &o, auto col) {
        constexpr int s = decltype(col)::value;
        if constexpr (s < S) {
            bf16x8 af[MI];
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) af[mi] = make_frag<2, 1, a_of(s), 0>(o.aw[mi]);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    union { u32x4 u; bf16x8 v; } bf;
                    bf.u = o.b[r][ni][b_of(s)];
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
                        acc[mi][ni][r * S + s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mi], bf.v, acc[mi][ni][r * S + s], 0, 0, 0);
                }
        }
    };
    auto mfma_step = [&](const Ops &o) {
        mfma_cols(o, std::integral_constant<int, 1>{});
        mfma_cols(o, std::integral_constant<int, 0>{});
        mfma_cols(o, std::integral_constant<int, 2>{});
    };
    // Interleaving hint for one step: after every MFMA one LDS read (while any are
    // left) and a few VALU instructions, so that the next step's operand requests,
    // the address arithmetic and the v_perm of the shifted fragments issue in the
    // shadow of the MFMAs instead of between two steps (one MFMA wave per SIMD:
    // nothing else would fill the gap).
    auto interleave = [&]() {
        constexpr int kMfma = MI * NI * T, kReads = MI * (S > 1 ? 2 : 1) + R * NI * NPH + 1;
#pragma unroll
        for (int i = 0; i < kMfma; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                 // MFMA
            if (i < kReads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); // DS read
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);                 // VALU
        }
    };
    // Requests the operands of segment `seg` of the rows at byte addresses ra / rx[]
    // into `o`.  `tail`: the segment is the last of its row, nothing lies right of it.
    const uint32_t astep = 64 * p.dy_ostride, xstep = 64 * p.x_cstride, pw = 2 * p.PW;
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    // have_blk0: the caller has filled blk[0] already (the block a step looks at to its right is
    // the next step's own block)
    auto request = [&](Ops &o, uint32_t ra, const uint32_t (&rx)[R], int seg, bool tail, bool have_blk0 = false) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            if (!(have_blk0 && S > 1)) o.aw[mi].blk[0] = lds16(ra + mi * astep + 16 * seg);
            if constexpr (S > 1) {
                // nothing lies right of a row's last segment.  Where the caller knows at compile
                // time that this is one, the block is a constant; otherwise it is read from the
                // zero row the dynamic LDS block starts with.
                if (__builtin_constant_p(tail) && tail) o.aw[mi].blk[1] = u32x4{0, 0, 0, 0};
                else o.aw[mi].blk[1] = lds16(tail ? lds0 : ra + mi * astep + 16 * seg + 16);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int ph = 0; ph < NPH; ++ph) o.b[r][ni][ph] = lds16(rx[r] + ni * xstep + ph * pw + 16 * seg);
    };
    auto compute = [&](uint32_t base) {
        // byte addresses in LDS of this lane's output channel / input channel
        const uint32_t ac = lds0 + 2 * (base + rows_elems + (wm * 32 * MI + l32) * p.dy_ostride);
        const uint32_t xc = lds0 + 2 * (base + rows_elems + TILE_O * p.dy_ostride + (wn * 32 * NI + l32) * p.x_cstride);
        const uint32_t tab = lds0 + 2 * base + half * 16; // row table, this half-wave's entries
        // the KS waves that share a tile take every KS-th row pair each
        const int nrp = p.LRpad / 2, segs = SC > 0 ? SC : p.SEGS;
        if constexpr (R == 1 && S == 1) {
            // One tap: a step is MI*NI MFMAs, far too short to hide the two LDS round trips behind
            // it (row table, then operands) when operands are asked for one step ahead -- counters
            // and timings showed the MFMA waves of these layers waiting on LDS four fifths of the
            // time.  Without a window no step depends on its neighbour, so: the KS waves take
            // every KS-th (row pair, segment) step, whatever the row (rows per chunk need not be a
            // multiple of 2*KS for all of them to work); operands are requested two steps ahead
            // into a ring of three sets, the row table three steps ahead.
            const int total = nrp * segs;
            if (ks >= total) return;
            const int n = (total - ks + KS - 1) / KS;
            // step index of this wave's i-th step, clamped: requests past the end re-read the last step
            auto entry_of = [&](int i) {
                const int t = min(ks + i * KS, total - 1);
                return lds16(tab + 32 * (int)fdiv(t, p.m_segs));
            };
            auto ask = [&](Ops &o, int i, const u32x4 &e) {
                const int t = min(ks + i * KS, total - 1);
                const int seg = t - (int)fdiv(t, p.m_segs) * segs;
                const uint32_t rxx[R] = {xc + 2 * e[1]};
                request(o, ac + 2 * e[0], rxx, seg, true);
            };
            Ops O0, O1, O2;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) O0.aw[mi].prev3 = O1.aw[mi].prev3 = O2.aw[mi].prev3 = 0;
            u32x4 e0 = entry_of(0), e1 = entry_of(1), e_ahead = entry_of(2);
            ask(O0, 0, e0);
            ask(O1, 1, e1);
            int i = 0;
#define CAC_PW_PHASE(USE, GET)                    \
    {                                             \
        const u32x4 e_now = e_ahead;              \
        e_ahead = entry_of(i + 3);                \
        ask(GET, i + 2, e_now);                   \
        mfma_step(USE);                           \
        interleave();                             \
        if (++i == n) break;                      \
    }
            for (;;) {
                CAC_PW_PHASE(O0, O2)
                CAC_PW_PHASE(O1, O0)
                CAC_PW_PHASE(O2, O1)
            }
#undef CAC_PW_PHASE
            return;
        }
        const int nsteps = ((nrp - ks + KS - 1) / KS) * segs;
        if (KS > 1 && nsteps == 0) return;

        // current rows of this lane and the raw table entry of the next row pair
        u32x4 e = lds16(tab + 32 * ks);
        uint32_t ra = ac + 2 * e[0], rx[R];
#pragma unroll
        for (int r = 0; r < R; ++r) rx[r] = xc + 2 * e[1 + r];
        u32x4 e_next = lds16(tab + 32 * min(ks + KS, nrp - 1));

        Ops X, Y;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) X.aw[mi].prev3 = 0;
        request(X, ra, rx, 0, segs == 1);

        if constexpr (SC > 0 && NPH == 1) {
            // Row pairs as an outer loop, the SC segments of a row unrolled.  The operand sets
            // alternate from step to step; an odd SC swaps their roles from one row to the next.
            int rp = ks;
            // step SGI of a row pair: MFMAs on USE while GET receives the operands of the next
            // step (one segment to the right, or the first segment of the wave's next row pair)
#define CAC_ROWSTEP(USE, GET, SGI)                                                                  \
    if constexpr (SGI < SC) {                                                                       \
        if constexpr (SGI + 1 < SC) {                                                               \
            _Pragma("unroll") for (int mi = 0; mi < MI; ++mi) {                                     \
                GET.aw[mi].prev3 = USE.aw[mi].blk[0][3];                                            \
                GET.aw[mi].blk[0] = USE.aw[mi].blk[1];                                              \
            }                                                                                       \
            request(GET, ra, rx, SGI + 1, SGI + 2 == SC, true);                                     \
        } else {                                                                                    \
            ra = ac + 2 * e_next[0];                                                                \
            _Pragma("unroll") for (int r = 0; r < R; ++r) rx[r] = xc + 2 * e_next[1 + r];           \
            e_next = lds16(tab + 32 * min(rp + 2 * KS, nrp - 1));                                   \
            _Pragma("unroll") for (int mi = 0; mi < MI; ++mi) GET.aw[mi].prev3 = 0;                 \
            request(GET, ra, rx, 0, SC == 1);                                                       \
            rp += KS;                                                                               \
        }                                                                                           \
        mfma_step(USE);                                                                             \
        interleave();                                                                               \
    }
#define CAC_ROW(A, B)                                                                              \
    CAC_ROWSTEP(A, B, 0) CAC_ROWSTEP(B, A, 1) CAC_ROWSTEP(A, B, 2) CAC_ROWSTEP(B, A, 3)            \
    CAC_ROWSTEP(A, B, 4) CAC_ROWSTEP(B, A, 5) CAC_ROWSTEP(A, B, 6) CAC_ROWSTEP(B, A, 7)
            static_assert(SC <= 8, "row steps are written out up to 8");
            const int nrows = nsteps / SC;
            if constexpr (SC % 2 == 0) {
                for (int i = 0; i < nrows; ++i) { CAC_ROW(X, Y) }
            } else {
                for (int i = 0;;) {
                    CAC_ROW(X, Y)
                    if (++i == nrows) break;
                    CAC_ROW(Y, X)
                    if (++i == nrows) break;
                }
            }
#undef CAC_ROW
#undef CAC_ROWSTEP
            return;
        }
        int seg = 0, rp = ks;
        // One step: MFMAs on USE, operands of the following step requested into GET
        // (same rows one segment to the right, or the next row pair, whose table
        // entry was requested a row pair ago).
#define CAC_STEP(USE, GET)                                                                        \
    if (seg + 1 < segs) {                                                                         \
        _Pragma("unroll") for (int mi = 0; mi < MI; ++mi) GET.aw[mi].prev3 = USE.aw[mi].blk[0][3]; \
        request(GET, ra, rx, seg + 1, seg + 2 == segs);                                           \
        mfma_step(USE);                                                                           \
        interleave();                                                                             \
        ++seg;                                                                                    \
    } else {                                                                                      \
        ra = ac + 2 * e_next[0];                                                                  \
        _Pragma("unroll") for (int r = 0; r < R; ++r) rx[r] = xc + 2 * e_next[1 + r];             \
        e_next = lds16(tab + 32 * min(rp + 2 * KS, nrp - 1));                   \
        _Pragma("unroll") for (int mi = 0; mi < MI; ++mi) GET.aw[mi].prev3 = 0;                   \
        request(GET, ra, rx, 0, segs == 1);                                                       \
        mfma_step(USE);                                                                           \
        interleave();                                                                             \
        seg = 0;                                                                                  \
        rp += KS;                                                                                 \
    }
        if constexpr (NPH == 1) {
            for (int t = 0;;) {
                CAC_STEP(X, Y)
                if (++t == nsteps) break;
                CAC_STEP(Y, X)
                if (++t == nsteps) break;
            }
        } else {
            // Two column phases double the xhat operands, and a second operand set does not fit the register file next to the
            // accumulators.  But a phase's operands are free as soon as its own columns are multiplied: the middle column is
            // all that phase 0 serves, so the next step's phase 0 and window are requested before the six MFMAs of the outer
            // columns, and its phase 1 after them, in front of the next middle column (418 -> 562 at 21 x 21, batch 236, tiles of 2:
            // 259 -> 234 us; layers that wait for their copy waves instead, 128 -> 256 at 28 x 28 uncompressed: 42.9 either way).
            for (int t = 0; t < nsteps; ++t) {
                mfma_cols(X, std::integral_constant<int, 1>{});
                Window<2> nw[MI];
                if (seg + 1 < segs) {
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) nw[mi].prev3 = X.aw[mi].blk[0][3];
                    ++seg;
                } else { // (past the last step: the last row pair again, for nobody)
                    ra = ac + 2 * e_next[0];
#pragma unroll
                    for (int r = 0; r < R; ++r) rx[r] = xc + 2 * e_next[1 + r];
                    e_next = lds16(tab + 32 * min(rp + 2 * KS, nrp - 1));
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) nw[mi].prev3 = 0;
                    seg = 0;
                    rp += KS;
                }
                const bool tail = seg + 1 == segs;
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) {
                    nw[mi].blk[0] = lds16(ra + mi * astep + 16 * seg);
                    nw[mi].blk[1] = lds16(tail ? lds0 : ra + mi * astep + 16 * seg + 16);
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) X.b[r][ni][0] = lds16(rx[r] + ni * xstep + 16 * seg);
                __builtin_amdgcn_sched_barrier(0);
                mfma_cols(X, std::integral_constant<int, 0>{});
                mfma_cols(X, std::integral_constant<int, 2>{});
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) X.b[r][ni][NPH - 1] = lds16(rx[r] + ni * xstep + (NPH - 1) * pw + 16 * seg);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) X.aw[mi] = nw[mi];
            }
        }
#undef CAC_STEP
    };

    __syncthreads(); // buffer 0 holds the first chunk
    uint32_t base = base0;
    for (int ci = ci_begin; ci < ci_end; ++ci) {
        compute(base);
        __syncthreads();
        base = base0 + base1 - base;
    }

    // ---- epilogue --------------------------------------------------------------------
    // accumulator register j of lane l holds row 8*(j/4) + 4*(l/32) + j%4, column l%32.
    // The accumulators are handled as G groups of 4 registers: g = (j/4)*(G/4) + (mi*NI + ni)*T + tap.
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    typedef f32x4 __attribute__((aligned(4))) f32x4_u;
    constexpr int G = MI * NI * T * 4;
    static_assert(KS == 1 || KS == 2 || KS == 4, "the K-split waves share the four row groups");
    static_assert(KS == 1 || T != 9 || MI * NI * (4 / KS) == 1, "a wave's groups are read before their place is used again");
    // The KS waves of a tile hold sums over different pixels.  They all leave them in LDS (the staging buffers
    // are dead: the loop above ends with a barrier), and wave ks adds up the groups with j/4 in [ks*4/KS, (ks+1)*4/KS): its own, then
    // the other waves', in wave order.  red[wm, wn][source wave][g][lane].  (Its own it could keep in registers, but which ones they
    // are depends on the wave: KS copies of all that follows, and the code of a kernel that goes through it once comes from memory.)
    f32x4 *red = (f32x4 *)smem + ((wn * WM + wm) * KS) * (G * 64) + lane;
#define CAC_G(mi, ni, t, jq) ((jq) * (G / 4) + ((mi) * NI + (ni)) * T + (t))
#define CAC_GROUP(mi, ni, t, jq) \
    f32x4 { acc[mi][ni][t][4 * (jq)], acc[mi][ni][t][4 * (jq) + 1], acc[mi][ni][t][4 * (jq) + 2], acc[mi][ni][t][4 * (jq) + 3] }
    if constexpr (KS > 1) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int jq = 0; jq < 4; ++jq) red[(ks * G + CAC_G(mi, ni, t, jq)) * 64] = CAC_GROUP(mi, ni, t, jq);
        __syncthreads();
    }
    // Output: dW itself (one slice), or this slice's partial sums in the workspace, in the same
    // [o][c][tap] order, so that the sum over the slices is a plain stream.
    float *out = p.direct ? p.out : p.out + (long)slice * p.K * p.C * T;
    const bool inside = o0 + TILE_O <= p.K && c0 + TILE_C <= p.C; // no edge of dW crosses the tile
    // Nine taps, a tile inside dW, rows of dW a multiple of 16 bytes: a group (8 output channels x
    // 32 input channels x 9 taps) is 8 contiguous runs of 1152 bytes in memory.  It goes through
    // a wave-private 9 KB of LDS, [row][c][tap], and leaves as 16-byte stores in which the lanes
    // of a wave cover whole runs (a lane's own 36-byte runs, unaligned and 36 bytes apart, cost
    // the store unit 1.5 us per group).  The 9 KB: with the pixels split over the waves, the part
    // of `red` that holds the wave's share of its own groups, which it has read by then and nobody else reads;
    // otherwise the dead staging buffers.
    const bool runs16 = T == 9 && inside && (p.C & 3) == 0;
    float *tb = KS > 1 ? (float *)((f32x4 *)smem + (((wn * WM + wm) * KS + ks) * G + (ks * 4 / KS) * (G / 4)) * 64)
                       : (float *)smem + wave * (8 * 32 * 9);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int jw = 0; jw < 4 / KS; ++jw) {
                const int jq = KS > 1 ? ks * (4 / KS) + jw : jw;
                f32x4 v[T];
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if constexpr (KS == 1) {
                        v[t] = CAC_GROUP(mi, ni, t, jw);
                    } else {
                        v[t] = red[(ks * G + CAC_G(mi, ni, t, jq)) * 64];
#pragma unroll
                        for (int k2 = 0; k2 < KS - 1; ++k2) v[t] += red[((k2 + (k2 >= ks)) * G + CAC_G(mi, ni, t, jq)) * 64];
                    }
                }
                if (T == 9 && runs16) {
#pragma unroll
                    for (int t = 0; t < T; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e) tb[half * 1152 + l32 * 9 + e * 288 + t] = v[t][e];
                    // (the wave reads what it wrote itself: LDS serves a wave's requests in order)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    const long row0 = (long)(o0 + (wm * MI + mi) * 32 + 8 * jq) * p.C + c0 + (wn * NI + ni) * 32;
#pragma unroll
                    for (int k = 0; k < 9; ++k) {
                        const int q4 = k * 64 + lane, rr = q4 / 72, w4 = q4 - rr * 72; // row, 16-byte unit of its run
                        *(f32x4 *)(out + (row0 + (long)rr * p.C) * 9 + 4 * w4) = ((const f32x4 *)tb)[q4];
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    continue;
                }
                // the T taps of one (o, c) are consecutive floats
                const int c = c0 + (wn * NI + ni) * 32 + l32;
                const int ob = o0 + (wm * MI + mi) * 32 + 8 * jq + 4 * half;
                float *dst = out + ((long)ob * p.C + c) * T;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (inside || (ob + e < p.K && c < p.C)) {
                        float *d = dst + (long)e * p.C * T;
                        if constexpr (T == 9) {
                            *(f32x4_u *)d = f32x4{v[0][e], v[1][e], v[2][e], v[3][e]};
                            *(f32x4_u *)(d + 4) = f32x4{v[4][e], v[5][e], v[6][e], v[7][e]};
                            d[8] = v[8][e];
                        } else {
#pragma unroll
                            for (int t = 0; t < T; ++t) d[t] = v[t][e];
                        }
                    }
                }
            }
#undef CAC_GROUP
#undef CAC_G
}

// The slice sum as a launch of its own (body and description: dw_reduce.h).
template <int SY, int V> __global__ void __launch_bounds__(256) dw_reduce_kernel(DwReduceTail t)
{
    __shared__ __align__(16) unsigned char red[SY > 1 ? 4096 : 16];
    dw_reduce_body<SY, V, 1>(t, blockIdx.x, 0, threadIdx.x, red);
}


// Kernel table: filter/stride family x workgroup shape.
struct Variant {
    int R, SG, MI, NI, WM, WN, KS;
    hipError_t (*launch)(const DwMfmaParams &, const RepackParams &, dim3, hipStream_t);
};

template <int R, int S, int SG, int PAD, int MI, int NI, int WM, int WN, int KS, int SC, bool DYL, int WIDEZ, int FL>
hipError_t launch_fixed(const DwMfmaParams &p, const RepackParams &rep, dim3 grid, hipStream_t st)
{
    auto kern = dw_mfma_kernel<R, S, SG, PAD, MI, NI, WM, WN, KS, SC, DYL, WIDEZ, FL>;
    // (per instantiation; once per process, whichever host thread comes first)
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); });
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL(kern, grid, dim3(128 * WM * WN * KS), p.lds_bytes, st, p, rep);
    return hipGetLastError();
}
// Picks the instantiation with the width of a pooling tile and, where there is one, the row length built in.
template <int R, int S, int SG, int PAD, int MI, int NI, int WM, int WN, int KS, int FL>
hipError_t launch_width(const DwMfmaParams &p, const RepackParams &rep, dim3 grid, hipStream_t st)
{
    if constexpr (S == 3 && SG == 1) {
        if constexpr (KS == 4) {
            if (p.dy_direct) {
                switch (p.SEGS) {
                case 1: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 1, true, 0, FL>(p, rep, grid, st);
                case 2: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 2, true, 0, FL>(p, rep, grid, st);
                case 4: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 4, true, 0, FL>(p, rep, grid, st);
                default: break;
                }
            }
        }
        if constexpr (FL == 0) {
            if (p.widez) {
                switch (p.SEGS) {
                case 1: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 1, false, 1, FL>(p, rep, grid, st);
                case 2: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 2, false, 1, FL>(p, rep, grid, st);
                case 4: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 4, false, 1, FL>(p, rep, grid, st);
                case 7: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 7, false, 1, FL>(p, rep, grid, st);
                default: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 0, false, 1, FL>(p, rep, grid, st);
                }
            }
        }
        switch (p.SEGS) {
        case 1: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 1, false, 0, FL>(p, rep, grid, st);
        case 2: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 2, false, 0, FL>(p, rep, grid, st);
        case 4: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 4, false, 0, FL>(p, rep, grid, st);
        case 7: return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 7, false, 0, FL>(p, rep, grid, st);
        default: break;
        }
    }
    if constexpr (S == 3 && SG == 2 && FL < 0) {
        if (p.widez == 2) return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 0, false, 2, FL>(p, rep, grid, st);
        if (p.widez) return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 0, false, 1, FL>(p, rep, grid, st);
    }
    return launch_fixed<R, S, SG, PAD, MI, NI, WM, WN, KS, 0, false, 0, FL>(p, rep, grid, st);
}
template <int R, int S, int SG, int PAD, int MI, int NI, int WM, int WN, int KS>
hipError_t launch_variant(const DwMfmaParams &p, const RepackParams &rep, dim3 grid, hipStream_t st)
{
    switch (p.kw_log2) {
    case 0: return launch_width<R, S, SG, PAD, MI, NI, WM, WN, KS, 1 - SG>(p, rep, grid, st);
    case 1: return launch_width<R, S, SG, PAD, MI, NI, WM, WN, KS, 2 - SG>(p, rep, grid, st);
    case 2: return launch_width<R, S, SG, PAD, MI, NI, WM, WN, KS, 3 - SG>(p, rep, grid, st);
    default: return launch_width<R, S, SG, PAD, MI, NI, WM, WN, KS, 4 - SG>(p, rep, grid, st);
    }
}

const Variant kVariants[] = {
    {3, 1, 1, 1, 2, 2, 1, launch_variant<3, 3, 1, 1, 1, 1, 2, 2, 1>}, // 3x3: 64 x 64 tile, 144 accumulators per wave
    {3, 1, 1, 1, 1, 1, 4, launch_variant<3, 3, 1, 1, 1, 1, 1, 1, 4>}, // 3x3: 32 x 32 tile, the pixels split over 4 waves
    {3, 2, 1, 1, 2, 2, 1, launch_variant<3, 3, 2, 1, 1, 1, 2, 2, 1>},
    {3, 2, 1, 1, 1, 1, 4, launch_variant<3, 3, 2, 1, 1, 1, 1, 1, 4>},
    {1, 1, 2, 2, 2, 2, 1, launch_variant<1, 1, 1, 0, 2, 2, 2, 2, 1>}, // 1x1: 128 x 128 tile
    {1, 1, 2, 2, 1, 1, 4, launch_variant<1, 1, 1, 0, 2, 2, 1, 1, 4>}, // 1x1:  64 x 64 tile, the pixels split over 4 waves
    {1, 1, 2, 2, 1, 1, 1, launch_variant<1, 1, 1, 0, 2, 2, 1, 1, 1>}, // 1x1:  64 x 64 tile, one wave
    {1, 2, 2, 2, 2, 2, 1, launch_variant<1, 1, 2, 0, 2, 2, 2, 2, 1>},
    {1, 2, 2, 2, 1, 1, 4, launch_variant<1, 1, 2, 0, 2, 2, 1, 1, 4>},
    {1, 2, 2, 2, 1, 1, 1, launch_variant<1, 1, 2, 0, 2, 2, 1, 1, 1>},
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

} // namespace

namespace {

// The plan for one entry of the kernel table; false when the geometry does not fit it.
bool plan_with(const Geom &g, int vi, int widez, DwMfmaPlan *plan)
{
    auto log2_of = [](int k) { return k == 1 ? 0 : k == 2 ? 1 : k == 4 ? 2 : k == 8 ? 3 : -1; };
    const int khl = log2_of(g.kh), kwl = log2_of(g.kw);
    const int T = g.R * g.S;
    const Variant &var = kVariants[vi];
    const int KS = var.KS;
    const int NT = 64 * var.WM * var.WN * KS;
    const int tile_o = 32 * var.MI * var.WM, tile_c = 32 * var.NI * var.WN;
    const int lds_budget = (NT == 256 ? 156 : NT == 128 ? 78 : 39) * 1024; // whole CU / half / quarter
    const int groups = var.MI * var.NI * T * 4;                             // accumulator groups of 4 per wave
    const int red_bytes = KS > 1 ? var.WM * var.WN * KS * groups * 64 * 16 : 0;

    DwMfmaParams base{};
    base.N = g.N; base.C = g.C; base.K = g.K; base.H = g.H; base.W = g.W; base.P = g.P; base.Q = g.Q;
    base.Hp = g.Hp; base.Wp = g.Wp;
    base.kh_log2 = khl; base.kw_log2 = kwl;
    base.widez = widez;
    base.SEGS = (g.Q + 7) / 8;
    base.Qpad = base.SEGS * 8;
    base.ZV = (g.Wp + 7) / 8;
    const int NPH = g.S == 1 ? 1 : g.sh;  // xhat column phases kept per row
    // width of one phase of an xhat row in LDS: the padded output row, or what the
    // staging of whole 8-value items writes if that is more
    const int f_log2 = kwl - (g.sh == 2 ? 1 : 0);
    base.PW = max(base.Qpad, f_log2 >= 0 ? (8 * base.ZV) << f_log2 : 4 * base.ZV);
    base.XW = NPH * base.PW;              // one xhat row in LDS: all phases
    base.tile_o = tile_o; base.tile_c = tile_c;

    auto pow2_at_least = [](int x) { int l = 2; while ((1 << l) < x) ++l; return l; };
    // Fills the chunk-dependent fields; false when the chunk does not fit the
    // per-thread copy registers or the LDS budget (two buffers).  `full`: nor does any longer one (its dY only grows).
    bool full = false;
    auto shape = [&](int nbi, int pr, DwMfmaParams &q) {
        q = base;
        q.NBI = nbi; q.PR = pr;
        q.LR = nbi * pr;
        q.LRpad = (q.LR + 1) & ~1;
        q.rowitems = q.LRpad * q.SEGS;
        q.ldy_log2 = pow2_at_least(q.rowitems); q.LDY = 1 << q.ldy_log2;
        full = q.LDY > NT || tile_o * q.LDY > NT * max_dy(widez);
        if (full) return false;
        q.dy_passes = (tile_o * q.LDY + NT - 1) / NT;
        q.RB = (g.P + pr - 1) / pr;
        if (!divides_exactly((uint64_t)((g.N + nbi - 1) / nbi) * q.RB, q.RB)) return false; // (a chunk's images and rows)
        int nz = 1;
        for (int rb = 0; rb < q.RB; ++rb) {
            const int p0 = rb * pr, p1 = min(p0 + pr, g.P) - 1;
            const int zlo = max(0, (p0 * g.sh - g.ph) >> khl);
            const int hhi = min(g.H - 1, p1 * g.sh + g.R - 1 - g.ph);
            nz = max(nz, (hhi >> khl) - zlo + 1);
        }
        q.NZ = nz;
        q.citems = nbi * nz * q.ZV;
        q.lpc_log2 = pow2_at_least(q.citems);   q.LPC = 1 << q.lpc_log2;
        q.z_passes = (tile_c * q.LPC + NT - 1) / NT;
        if (q.LPC > NT || q.z_passes > max_z(widez)) return false;
        if ((tile_o * q.LDY) % NT || (tile_c * q.LPC) % NT) return false; // passes cover the tile exactly
        // strides: an odd number of 16-byte units so that the 32 lanes of a half
        // wave (one output channel / input channel each) read distinct LDS banks
        q.dy_ostride = 8 * ((q.rowitems + 1) | 1); // + one block: the dY window looks one block past a row
        q.x_cstride = 8 * (((nbi * nz + 1) * (q.XW / 8)) | 1); // + the zero slot
        q.dy_direct = var.R == 3 && var.SG == 1 && var.KS == 4 && // (the kernels that exist with it: see launch_variant)
                      g.Q % 8 == 0 && q.rowitems == 64 && q.LDY == 64 && q.dy_passes == 8 && (q.SEGS == 1 || q.SEGS == 2 || q.SEGS == 4);
        q.lds_bytes = (q.XW + 2 * (q.LRpad * 8 + tile_o * q.dy_ostride + tile_c * q.x_cstride)) * 2;
        if (q.lds_bytes > lds_budget) return false;
        q.lds_bytes = max(q.lds_bytes, red_bytes); // the cross-wave sum reuses the staging space
        q.lds_bytes = max(q.lds_bytes, var.WM * var.WN * 8 * 32 * 9 * 4); // so does the epilogue's transpose (9 KB per wave)
        return true;
    };
    // Candidates: part of one image (nbi = 1, pr <= P) or several whole images.
    // Cost = MFMA steps spent per useful pixel row, then prefer longer chunks.
    DwMfmaParams best{};
    double best_cost = 1e30;
    auto consider = [&](int nbi, int pr) {
        DwMfmaParams q;
        if (!shape(nbi, pr, q)) return;
        const int rp_wave = (q.LRpad / 2 + KS - 1) / KS;                 // row pairs of the busiest wave
        const double steps = (double)q.RB * rp_wave * KS * q.SEGS;       // per group of nbi images
        const double useful = (double)nbi * g.P * g.Q / 16.0;
        const double per_chunk = rp_wave * q.SEGS;
        const double cost = steps / useful * (1.0 + 1.5 / per_chunk);     // barrier + refill share
        if (cost < best_cost) { best_cost = cost; best = q; }
    };
    for (int pr = 1; pr <= g.P && !full; ++pr) consider(1, pr);
    for (int nbi = 2; nbi <= min(g.N, 64) && !full; ++nbi) consider(nbi, g.P);
    if (best_cost > 1e29) return false;

    DwMfmaParams &p = plan->p;
    p = best;
    p.m_segs = magic_of(p.SEGS);
    p.m_pr = magic_of(p.PR);
    p.m_zv = magic_of(p.ZV);
    p.m_nz = magic_of(p.NZ);
    p.m_rb = magic_of(p.RB);

    p.tiles_o = (g.K + tile_o - 1) / tile_o;
    p.tiles_c = (g.C + tile_c - 1) / tile_c;
    const int ntiles = p.tiles_o * p.tiles_c;
    p.nchunks = ((g.N + p.NBI - 1) / p.NBI) * p.RB;
    // one workgroup per 256 threads of the 256 CUs, each with at least two chunks
    const int wg_target = 256 * (256 / NT);
    int want = max(1, wg_target / ntiles);
    want = min(want, max(1, p.nchunks / 2));
    p.chunks_per_slice = (p.nchunks + want - 1) / want;
    p.nslices = (p.nchunks + p.chunks_per_slice - 1) / p.chunks_per_slice;
    p.total_wg = p.nslices * ntiles;
    p.direct = p.nslices == 1;
    plan->grid = ((p.total_wg + 7) / 8) * 8;
    plan->threads = NT;
    plan->partial_bytes = p.direct ? 0 : (size_t)p.nslices * g.K * g.C * T * sizeof(float);
    plan->variant = vi;
    return true;
}

// Workgroup shape.  Splitting the pixels over the waves of a workgroup (KS > 1) cuts the
// partial sums a workgroup writes by KS at the price of shorter runs between barriers and
// twice the staging work per MFMA; it pays when a workgroup has only a few chunks to go
// through.  Among the others: the large tile unless it would be mostly padding.
bool plan_shape(const Geom &g, int widez, DwMfmaPlan *plan)
{
    DwMfmaPlan whole, split;
    bool have_whole = false, have_split = false;
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = kVariants[i];
        if (v.R != g.R || v.SG != g.sh) continue;
        const int to = 32 * v.MI * v.WM, tc = 32 * v.NI * v.WN;
        if (to > 64 && (g.K <= to / 2 || g.C <= tc / 2)) continue;
        if (v.KS > 1) {
            if (!have_split) have_split = plan_with(g, i, widez, &split);
        } else {
            if (!have_whole) have_whole = plan_with(g, i, widez, &whole);
        }
    }
    if (!have_whole && !have_split) return false;
    const int thr = g.R == 1 ? 12 : 24; // measured break-even (chunks per workgroup: split wins at 16, loses at 32)
    bool use_split = have_split && (!have_whole || split.p.chunks_per_slice <= thr);
#ifdef CAC_TUNING // development builds: CAC_DW_SHAPE=whole|split overrides the rule
    if (const char *f = getenv("CAC_DW_SHAPE")) {
        if (f[0] == 'w' && have_whole) use_split = false;
        if (f[0] == 's' && have_split) use_split = true;
    }
#endif
    *plan = use_split ? split : whole;
    return true;
}

} // namespace

bool dw_mfma_plan(const Geom &g, int dtype, DwMfmaPlan *plan)
{
    if (dtype != CAC_BF16) return false;
    if (g.R != g.S || g.sh != g.sw || g.ph != g.pw) return false;
    const bool f3 = g.R == 3 && g.ph == 1, f1 = g.R == 1 && g.ph == 0;
    if (!(f3 || f1) || (g.sh != 1 && g.sh != 2)) return false;
    auto log2_of = [](int k) { return k == 1 ? 0 : k == 2 ? 1 : k == 4 ? 2 : k == 8 ? 3 : -1; };
    const int khl = log2_of(g.kh), kwl = log2_of(g.kw);
    if (khl < 0 || kwl < 0) return false;
    if (g.Q > 256 || g.W > 1024) return false;
    // buffer loads address with 32-bit byte offsets and use 2^31 as "no load"
    if ((long)g.N * g.K * g.P * g.Q >= (1L << 30) || (long)g.N * g.C * g.Hp * g.Wp >= (1L << 30)) return false;

    // The split of the copy registers.  Of 200 random uncompressed layers the first split towards Z took 0.6 of the time from 48
    // chunks of the usual length per workgroup on, 0.75 from 24, 0.85 from 12, 0.89 (at most 0.91) from 8 and 1.02 (up to 1.44)
    // below four (128 -> 256 at 28 x 28, batch 128, 56 of them: 66 -> 47 us, 20 -> 76 at 4 x 4, batch 121, two: 15.7 -> 19.3).  The
    // second pays where it halves the chunks -- two rows of a wide map instead of one, no half-empty row pair -- and a workgroup
    // has many (64 -> 128 at 56 x 56, batch 128: 50.3 -> 43.6; 224 -> 272 at 36 x 53, batch 97: 213 -> 163; a fifth fewer chunks 120 -> 140;
    // few chunks up to 1.3 times the time).  Where only a split fits -- long rows -- the kernel of dw_tiled.hip is the other choice:
    // four times as slow in the mean, but 12.4 against 19.3 us for 9 -> 9 at 82 x 82, batch 1.
    //
    // Under stride 1 a chunk of output rows needs two Z rows more than it has, and the usual split leaves half its loads of dY
    // empty.  The first split is taken where it saves a quarter of the chunks, those of every tile counted: 102 of 400 random layers,
    // 0.60 of the time, the worst 0.98 (112 -> 112 at 56 x 56, batch 93: 175 -> 83 us); up to a quarter fewer 0.94 and at most
    // 1.13, more chunks 1.12 and up to 1.8.  On rows of 81 to 128 pixels only this split fits: 39 random layers 0.09 to 0.82 of the time of
    // dw_tiled.hip (192 -> 96 at 88 x 88, batch 28: 2002 -> 194 us).
    const bool may_widen = f3 && g.kw == 1;
#ifdef CAC_TUNING
    if (const char *f = getenv("CAC_DW_WIDE"); f && atoi(f) == 0) return plan_shape(g, 0, plan);
#endif
    if (!plan_shape(g, 0, plan))
        return may_widen && 2.0 * g.N * g.P * g.Q * (double)g.K * g.C * 9 >= 1e8 && plan_shape(g, 1, plan);
    if (!may_widen) return true;
    const auto work = [](const DwMfmaPlan &a) { return (double)a.p.nchunks * a.p.tiles_o * a.p.tiles_c; };
    if (g.sh == 1) {
        DwMfmaPlan wide;
        if (plan_shape(g, 1, &wide) && 4 * work(wide) <= 3 * work(*plan)) *plan = wide;
        return true;
    }
    if (plan->p.chunks_per_slice < 8) return true;
    const int usual = plan->variant;
    const auto small_tile = [](const DwMfmaPlan &a) { return kVariants[a.variant].KS > 1; };
    for (int w = 1; w <= 2; ++w) {
        if (w == 2 && plan->p.chunks_per_slice < 24) break;
        DwMfmaPlan wide;
        bool have = plan_shape(g, w, &wide);
        // The rule between the tiles counts chunks of the usual length: what it gives the large tile stays there.  Nor does
        // the second split leave the first one's large tile, which it does not fit on rows past 64, for a small one that has
        // more to copy, a chunk of every tile counted: 354 -> 823 at 94 x 94, batch 12, tiles of 2 x 1, has four times the tiles
        // for half the chunks, 325 against 776 us; 15 -> 10 at 112 x 112, batch 382, one tile either way, 161 against 76.  (Of 704
        // layers whose plan a split changes the 146 that this keeps on the large tile take 0.64 of the small one's time,
        // one of them more than 1.05.)
        const bool shrinks = have && !small_tile(*plan) && small_tile(wide);
        if (shrinks && (kVariants[usual].KS == 1 || work(wide) > 1.1 * work(*plan)))
            have = plan_with(g, plan->variant, w, &wide);
        // Below twelve chunks the first split pays by longer chunks alone, and in the same tile: tall pooling tiles leave few Z
        // items, so that the copy registers of dY bound a chunk and the split shortens it (3 -> 536 at 18 x 18, batch 421, tiles
        // of 8 x 1, nine chunks to a workgroup of the small tile, thirty of the large one: 38 against 54 us).
        const bool few = w == 1 && plan->p.chunks_per_slice < 12;
        if (few && have && wide.variant != usual) have = plan_with(g, usual, w, &wide);
        if (have && (w == 1 ? !few || wide.p.nchunks < plan->p.nchunks : 20L * wide.p.nchunks <= 11L * plan->p.nchunks)) *plan = wide;
        else break;
    }
    return true;
}

hipError_t launch_dw_reduce(const DwReduceTail &t, hipStream_t st)
{
    if (!t.blocks) return hipSuccess;
#define CAC_REDUCE(SY, V) hipLaunchKernelGGL((dw_reduce_kernel<SY, V>), dim3(t.blocks), dim3(256), 0, st, t)
    if (t.V == 4) {
        if (t.SY == 16) CAC_REDUCE(16, 4);
        else if (t.SY == 4) CAC_REDUCE(4, 4);
        else CAC_REDUCE(1, 4);
    } else {
        if (t.SY == 16) CAC_REDUCE(16, 1);
        else if (t.SY == 4) CAC_REDUCE(4, 1);
        else CAC_REDUCE(1, 1);
    }
#undef CAC_REDUCE
    return hipGetLastError();
}

// LDS of the kernel, in elements (all multiples of 8): a staging buffer, and what laying out a block of the filter takes; the waves
// that do so in the part of a buffer that holds dY, or four past both buffers where that has no room for two.
static int buffer_elems(const DwMfmaParams &p) { return p.LRpad * 8 + p.tile_o * p.dy_ostride + p.tile_c * p.x_cstride; }
static int repack_elems(const FilterRepack &f) { return 16 * (32 * f.RS + 2); }
static bool repack_past(const DwMfmaParams &p, const FilterRepack &f) { return p.tile_o * p.dy_ostride < 2 * repack_elems(f); }
static int repack_waves(const DwMfmaParams &p, const FilterRepack &f) { return repack_past(p, f) ? 4 : min(4, p.tile_o * p.dy_ostride / repack_elems(f)); }

// Whether the kernel's launch has room for the data gradient's repacks, which cost 4-10 us in one of their own.
// 1: with 64 compute units and more to spare, in workgroups of their own there (18 random layers: 0.62-0.93 of the backward pass).
// 2: a filter of 256 blocks and more, read in 16-byte pieces: every MFMA wave lays out two of them at most while it waits for its
// first chunk (66 random layers: 0.962 of the backward pass, none over 1.02; 512 -> 2048, 1 x 1 at 7 x 7, batch 64: 43.8 -> 40.7 us, 512 ->
// 512, 3 x 3 at 7 x 7, batch 256: 1 to 4 %).
// Else neither: smaller filters and element-wise ones delay the waves that have a block by 4-6 us (224 -> 32, 1 x 1 at 34 x 34, batch 93,
// 41.0 -> 43.6), and workgroups behind 256 of the kernel's are a tail as long as the launch.
int dw_takes_repack(const DwMfmaPlan &plan, const RepackParams &rep)
{
    const DwMfmaParams &p = plan.p;
    const FilterRepack &f = rep.f;
    if (plan.threads != 256) return 0;
    if (plan.grid <= 192) return 1;
    const int blocks = (int)f.blocks();
    if (rep.in_blocks || rep.zero_n || blocks < 256 || blocks > 2 * repack_waves(p, f) * p.total_wg || f.Cw % 32 || f.Cw * f.RS % 8) return 0;
    return repack_past(p, f) && 2 * (p.XW + 2 * buffer_elems(p) + 4 * repack_elems(f)) > 160 * 1024 ? 0 : 2;
}

// `defer`: when given, the slice sum is not launched; what it has to do is written there instead
// (blocks = 0 when the main kernel has written dW itself) and the caller sees to it.
// `rep`: repacks for the same launch; *rep_done says whether it has taken them.
hipError_t launch_dw_mfma(const DwMfmaPlan &plan, const void *Z, const void *dY, float *dW, void *ws, hipStream_t st,
                          DwReduceTail *defer, const RepackParams *rep, bool *rep_done)
{
    DwMfmaParams p = plan.p;
    p.Z = (const bf16_t *)Z;
    p.dY = (const bf16_t *)dY;
    p.out = p.direct ? dW : (float *)ws;
    p.own_wgs = plan.grid;
    if (defer) defer->blocks = 0;
    const Variant &var = kVariants[plan.variant];
    RepackParams r{};
    unsigned more = 0;
    switch (rep ? dw_takes_repack(plan, *rep) : 0) {
    case 1:
        r = *rep;
        r.in_blocks = (r.in_blocks + 1) & ~1; // (two blocks to a workgroup, both of a kind: the same barriers)
        more = (r.blocks() + 1) / 2;
        *rep_done = true;
        break;
    case 2:
        r = *rep;
        p.rep_waves = repack_waves(p, r.f);
        p.rep_blocks = (int)r.f.blocks();
        p.rep_elems = repack_elems(r.f);
        p.rep_at = repack_past(p, r.f) ? p.XW + 2 * buffer_elems(p) : p.XW + buffer_elems(p) + p.LRpad * 8;
        if (repack_past(p, r.f)) p.lds_bytes = max(p.lds_bytes, 2 * (p.XW + 2 * buffer_elems(p) + 4 * p.rep_elems));
        *rep_done = true;
        break;
    }
    hipError_t e = var.launch(p, r, dim3(plan.grid + more), st);
    if (e != hipSuccess || p.direct) return e;
    const DwReduceTail t = make_reduce_tail((const float *)ws, dW, (long)p.K * p.C * var.R * var.R, p.nslices);
    if (defer) {
        *defer = t;
        return hipSuccess;
    }
    return launch_dw_reduce(t, st);
}

} // namespace cac
