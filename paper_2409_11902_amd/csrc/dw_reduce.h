// Sum of the weight gradient's partial sums over the pixel slices (second step of the split
// weight-gradient kernel, see dw_mfma.hip), as a device function so that the launch can be shared
// with other small work of a backward pass.
#pragma once
#include "common.h"

namespace cac {

// What is left to do after the main weight-gradient kernel when its reduction is deferred.
struct DwReduceTail {
    const float *part; // [nslices][total] partial sums
    float *dW;
    long total;        // elements of dW
    int nslices;
    int SY, V;         // thread rows over the slices; floats per vector
    unsigned blocks;   // blocks of 256 threads; 0: nothing to do
};

// Vectors of 4 floats when a slice is a whole number of them (every slice then starts aligned);
// thread rows over the slices when there are many of them.
inline DwReduceTail make_reduce_tail(const float *part, float *dW, long total, int nslices)
{
    DwReduceTail t{part, dW, total, nslices, 1, 1, 0};
    t.V = total % 4 == 0 ? 4 : 1;
    t.SY = nslices >= 32 ? 16 : nslices >= 8 ? 4 : 1;
    t.blocks = (unsigned)((total / t.V + 256 / t.SY - 1) / (256 / t.SY));
    return t;
}

// dW = sum over the slices of their partial sums, in slice order.  256 threads (tid) own 256/SY vectors of V floats to a block;
// their SY thread rows take every SY-th slice each and are combined through LDS (4 KB at red) in a fixed order, so the result
// does not depend on scheduling, nor on the launch it runs in.  NB blocks at once, `step` apart (one past the last: no column).
template <int SY, int V, int NB>
__device__ __forceinline__ void dw_reduce_body(const DwReduceTail &t, unsigned block, unsigned step, int tid, void *red_lds)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    constexpr int CX = 256 / SY;
    const int nslices = t.nslices, cx = tid % CX, sy = tid / CX;
    vec *red = (vec *)red_lds;
    const long nvec = t.total / V;
    const vec *src[NB];
    bool valid[NB];
    vec sum[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const long col = (long)(block + b * step) * CX + cx;
        valid[b] = col < nvec;
        src[b] = (const vec *)t.part + (valid[b] ? col : 0);
        sum[b] = 0.f;
    }
    int sl = sy;
    for (; sl + 3 * SY < nslices; sl += 4 * SY) {
        vec v[NB][4];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[b][k] = src[b][(long)(sl + k * SY) * nvec];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) sum[b] += v[b][k];
    }
    for (; sl < nslices; sl += SY)
#pragma unroll
        for (int b = 0; b < NB; ++b) sum[b] += src[b][(long)sl * nvec];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (SY > 1) {
            if (b) __syncthreads();
            red[sy * CX + cx] = sum[b];
            __syncthreads();
            if (sy == 0)
#pragma unroll
                for (int k = 1; k < SY; ++k) sum[b] += red[k * CX + cx];
        }
        if (valid[b] && sy == 0) ((vec *)t.dW)[(long)(block + b * step) * CX + cx] = sum[b];
    }
}

// The slice sum in the workgroups of another kernel's launch: workgroup `wg` of `nwg`, of 256 or 512 threads, few of which a compute
// unit holds (that kernel's registers and LDS): four blocks at once, sixteen loads of a thread in flight.
template <int SY, int V> __device__ __forceinline__ void dw_reduce_share_by(const DwReduceTail &t, unsigned wg, unsigned nwg, unsigned char *lds)
{
    constexpr int NB = V == 4 ? 4 : 1;
    const int tid = threadIdx.x & 255, sub = threadIdx.x >> 8, subs = blockDim.x >> 8;
    for (unsigned u = wg; u * subs < t.blocks; u += NB * nwg) {
        dw_reduce_body<SY, V, NB>(t, u * subs + sub, nwg * subs, tid, lds + sub * 4096);
        if (SY > 1) __syncthreads(); // (the next block's rows go to the same place)
    }
}
__device__ __forceinline__ void dw_reduce_share(const DwReduceTail &t, unsigned wg, unsigned nwg, unsigned char *lds)
{
    if (t.V == 4) {
        if (t.SY == 16) dw_reduce_share_by<16, 4>(t, wg, nwg, lds);
        else if (t.SY == 4) dw_reduce_share_by<4, 4>(t, wg, nwg, lds);
        else dw_reduce_share_by<1, 4>(t, wg, nwg, lds);
    } else {
        if (t.SY == 16) dw_reduce_share_by<16, 1>(t, wg, nwg, lds);
        else if (t.SY == 4) dw_reduce_share_by<4, 1>(t, wg, nwg, lds);
        else dw_reduce_share_by<1, 1>(t, wg, nwg, lds);
    }
}

// dw_mfma.hip: the reduction as a launch of its own.
hipError_t launch_dw_reduce(const DwReduceTail &t, hipStream_t st);

} // namespace cac
