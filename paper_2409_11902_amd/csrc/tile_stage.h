// What the kernels of conv_tile.hip and conv_dx2.hip share: staging of a channels-last input patch in LDS by all four
// waves of a workgroup, from a tensor that is read where it lies ([N][C][H][W], rows of any length).
#pragma once
#include "common.h"
#include "conv_mfma.h"

namespace cac {
namespace tile {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
constexpr uint32_t kNoLoad = 0x80000000u;
constexpr uint32_t kNoElem = 0x40000000u;
constexpr uint32_t kFrag = 64 * 16; // bytes of one fragment of the repacked filter

__device__ __forceinline__ uint32_t fdiv(uint32_t x, uint32_t magic) { return magic ? __umulhi(x, magic) : x; }
typedef __attribute__((address_space(3))) u32x4 *lds_u32x4_ptr;
typedef __attribute__((address_space(3))) u32x2 *lds_u32x2_ptr;
typedef __attribute__((address_space(3))) uint32_t *lds_u32_ptr;
typedef __attribute__((address_space(3))) uint16_t *lds_u16_ptr;
__device__ __forceinline__ u32x4 lds16(uint32_t addr) { return *(lds_u32x4_ptr)(uintptr_t)addr; }

// Keeps the compiler from computing what follows from `x` ahead of this point (and outside of loops).
__device__ __forceinline__ void opaque(uint32_t &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void opaque_s(uint32_t &x) { asm volatile("" : "+s"(x)); }

constexpr int kDumpBytes = 256 * 16; // past the buffers: 16 bytes for every lane of a workgroup

// A stage is KC channels of the patch, IPT images of PH x PWd pixels, in LDS as [pixel][KC + 8] elements.  An item is 8
// channels x GW pixels of one patch row: GW = 8, or 7 for rows of odd length (an item that starts on an odd element is
// read from the dword below, whose eight elements hold seven of the item).  A thread moves ITEMS items of a stage in
// parts of CB channels, one after the other through the same registers.  Pixels outside the image are never written:
// both buffers start as zeros.
template <int ITEMS, int GW, int KC, int CB = 4> struct PatchStage {
    static constexpr int KCS = KC + 8;      // an odd number of 16-byte units
    static constexpr int OCT = KC / 8;
    uint32_t e0[ITEMS], l0[ITEMS], m8[ITEMS];
    u32x4 r[ITEMS][CB];
    uint32_t par, plane, dump;
    int co, n_base, KCin;
    rsrc_t rs_in;

    __device__ __forceinline__ void init(const GatherParams &p, uint32_t lds0, uint32_t dump_base, int n_first, int hin0)
    {
        const int tid = threadIdx.x, win0 = p.dwmin, GX = p.GX, nitems = p.IPT * p.PH * GX * OCT;
        co = tid & (OCT - 1);
        n_base = n_first;
        KCin = p.KCin;
        plane = (uint32_t)p.Hin * p.Win;
        par = 0;
        dump = dump_base + tid * 16;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int it = tid + 256 * q;
            const int rest = it / OCT;
            const int rows = fdiv(rest, p.m_gx), gx = rest - rows * GX;
            const int g = fdiv(rows, p.m_ph), pr = rows - g * p.PH;
            const int hin = hin0 + pr, w0 = gx * GW;
            const bool ok = (it < nitems) & (hin >= 0) & (hin < p.Hin) & (n_base + g < p.N);
            uint32_t m = 0;
#pragma unroll
            for (int k = 0; k < GW; ++k) {
                const int w = w0 + k;
                m |= (ok & (w < p.Win) & (w >= win0) & (w < win0 + p.PWd)) ? 1u << k : 0u;
            }
            m8[q] = m;
            e0[q] = ok ? (uint32_t)((g * KCin + co * 8) * p.Hin + hin) * p.Win + w0 : kNoElem;
            l0[q] = lds0 + (uint32_t)(((g * p.PH + pr) * p.PWd + (w0 - win0)) * KCS + co * 8) * 2u;
        }
        rs_in = make_rsrc(p.in, (uint32_t)p.N * KCin * plane * 2u);
    }
    // loads of part h of stage s (past the last stage: nothing)
    __device__ __forceinline__ void fetch(int s, int h)
    {
        const uint32_t sbase = (uint32_t)(n_base * KCin + s * KC + CB * h) * plane;
        const int nvalid = KCin - (s * KC + co * 8 + CB * h); // channels of this lane's items that exist
        if (GW == 7) par = sbase & 1u;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            uint32_t e = e0[q] + sbase; // (no item: still far outside the tensor)
            opaque(e); // (the addresses of the stages are not to be kept in registers)
#pragma unroll
            for (int i = 0; i < CB; ++i) {
                const uint32_t ei = i < nvalid ? e : kNoElem;
                r[q][i] = __builtin_amdgcn_raw_buffer_load_b128(rs_in, (GW == 7 ? ei & ~1u : ei) * 2u, 0, 0);
                e += plane;
            }
        }
    }
    // rows that were read from the dword below an odd element: down by one element
    __device__ __forceinline__ void align_rows()
    {
        if constexpr (GW == 7) {
#pragma unroll
            for (int q = 0; q < ITEMS; ++q)
#pragma unroll
                for (int i = 0; i < CB; ++i) {
                    const uint32_t sh = ((e0[q] + par + i * plane) & 1u) * 16u;
                    u32x4 v = r[q][i];
                    v[0] = __builtin_amdgcn_alignbit(v[1], v[0], sh);
                    v[1] = __builtin_amdgcn_alignbit(v[2], v[1], sh);
                    v[2] = __builtin_amdgcn_alignbit(v[3], v[2], sh);
                    v[3] = v[3] >> sh;
                    r[q][i] = v;
                }
        }
    }
    // pixel px of the items, part h, to the buffer at offset buf
    __device__ __forceinline__ void put_px(uint32_t buf, int h, int px)
    {
        if (px >= GW) return;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            uint32_t v[CB / 2]; // half px%2 of dword px/2 of every row
#pragma unroll
            for (int k = 0; k < CB / 2; ++k) {
                const uint32_t lo = r[q][2 * k][px / 2], hi = r[q][2 * k + 1][px / 2];
                v[k] = (px & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
            }
            // (a pixel that is not wanted goes to a place of the lane's own past the buffers: no branch)
            const uint32_t a = (m8[q] & (1u << px)) ? l0[q] + buf + (px * (KCS * 2) + 2 * CB * h) : dump;
            if constexpr (CB == 8) *(lds_u32x4_ptr)(uintptr_t)a = u32x4{v[0], v[1], v[2], v[3]};
            else *(lds_u32x2_ptr)(uintptr_t)a = u32x2{v[0], v[1]};
        }
    }
    // both buffers zero, the first stage in buffer 0
    __device__ __forceinline__ void start(uint32_t lds0, uint32_t buf_bytes)
    {
#pragma unroll
        for (int h = 0; h < 8 / CB; ++h) {
            fetch(0, h);
            if (h == 0) {
                for (uint32_t i = threadIdx.x; i < 2 * buf_bytes / 16; i += 256) *(lds_u32x4_ptr)(uintptr_t)(lds0 + 16 * i) = u32x4{0, 0, 0, 0};
                __syncthreads(); // (the zeros of one thread lie where another writes pixels)
            }
            align_rows();
#pragma unroll
            for (int px = 0; px < GW; ++px) put_px(0, h, px);
        }
        __syncthreads();
    }
};

} // namespace tile
} // namespace cac
