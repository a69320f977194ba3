// Forward convolution / data gradient as an MFMA gather GEMM (see conv_mfma.hip).
#pragma once
#include "common.h"
#include "dw_reduce.h"
#include "filter_repack.h"

namespace cac {

struct GatherParams {
    const bf16_t *in;   // [N][Hin][Win][KCp], channels last; with nchw: the caller's tensor itself, [N][KCin][Hin][Win]
    const bf16_t *wt;   // [ntaps_total][KCp/16][Mp/32][64][8], MFMA fragment order
    const bf16_t *bias; // [M] or null
    bf16_t *out;        // [N][M][Hout][Wout]
    float *part;        // [ksplit][N][M][Hout*Wout] float sums when the channels are shared out, else null
    int tail_wgs;       // workgroups after the launch's own that add a weight gradient's slices (share_grid); up here, in a line
                        // that every kernel reads first: at the end of this record it was a cache miss of its own ahead of
                        // everything, 0.5 us of a launch
    int gx, gy, gz;     // the launch's own workgroups
    int N, M, Mp, KCp;
    int Hin, Win, Hout, Wout;
    int Hc, Wc;         // grid of output pixels of this launch: (h, w) = (i*os + a0, j*os + b0)
    int os, a0, b0, is; // input pixel of tap t: (i*is + dh[t], j*is + dw[t])
    int ntaps, ntaps_total;
    int dh[9], dw[9], wtap[9];
    int dhmin, dwmin;
    int PH, PWd;        // input patch of one image staged per workgroup (rows, columns)
    int IPT, patch_px;  // images per pixel tile; patch pixels of the whole tile
    int tiles_per_img, ngrp, gpw, nkb; // tiles per image; image groups; groups per workgroup; channel blocks
    int ksplit, kbs;    // workgroups sharing one tile's channel blocks (grid z); channel blocks of each
    int T, t_log2, kcs; // 32-channel groups staged per pass (1, 2 or 4; more than one only where taps * T is 4 or 8);
                        // LDS elements per patch pixel (32 * T + 8); a "channel block" above is 32 * T channels
    int nchw, KCin;     // the kernel reads the input in its own layout (KCin channels) instead of a channels-last copy
    int wide_store;     // the epilogue writes 16-byte runs of 8 pixels (whole planes, a multiple of 8 pixels each)
    int decim;          // forward, 1 x 1 filter, stride 2: `in` holds only the pixels the filter reaches (every second
                        // one of every second row), as an image of half the extent read with stride 1
    uint32_t m_wc, m_ppi, m_pwd, m_kbs, m_img; // division magics of Wc, Hc*Wc, PWd, kbs, PH*PWd
    uint32_t m_gx, m_ph;                       // ... of the 8-pixel groups of an input row and of PH (in-place copy)
    // conv_tile.hip
    int tile;           // the launch runs there (2: in conv_dx2.hip, 3: in conv_pw.hip, 4, 5: in conv_wave.hip)
    int gw, GX;         // pixels of a staged item; items of an input row
    int store_px;       // pixels per store of the epilogue: 8, 4, 2 or 1
    int buf_bytes, lds_bytes; // a staging buffer; all of the workgroup's LDS
    // conv_wave.hip
    int VH, IR;         // rows of LDS that an image takes; image rows staged per tile
    int mtiles;         // blocks of output channels
    // conv_pw.hip
    bf16_t *Z;          // the input's 2 x 2 mean record, written on the way, or null
    int pw_pool;        // the launch can form that record
    int tile_px;        // pixels of a tile
    int w_direct;       // the filter fragments are read from W itself ([M][KCin])
    uint32_t w_kstep, w_bytes; // bytes from one 16-channel step of the filter to the next; of all of it
    uint32_t m_w2;      // division magic of two image rows
    uint32_t wofs[9], toff[9]; // per tap: byte offset of its filter fragments; LDS byte offset within the patch
    DwReduceTail tail; // a weight gradient's slice sum in workgroups of this launch (share_grid)
};

// A data gradient's launch has workgroups to add the slices of the same layer's weight gradient: the sum is bound by memory
// where the launch is bound by the matrix cores or by latency, and a launch of its own costs 4 us and more.  They come after
// the launch's own, in the room that its last round leaves (in turns with them the sum's workgroups took the places of
// partners: 512 -> 512 at 14 x 14, batch 256, 14 us more than after them).
inline dim3 share_grid(GatherParams &p, dim3 grid, int threads)
{
    p.gx = grid.x; p.gy = grid.y; p.gz = grid.z;
    p.tail_wgs = 0;
    if (!p.tail.blocks) return grid;
    const unsigned subs = threads / 256, want = (p.tail.blocks + subs - 1) / subs;
    p.tail_wgs = want < 512 ? want : 512;
    return dim3(grid.x * grid.y * grid.z + p.tail_wgs);
}
// The workgroup's place in the launch's own grid; false when it had slices to add (done then).
__device__ __forceinline__ bool conv_block(const GatherParams &p, unsigned char *lds, unsigned &bx, unsigned &by, unsigned &bz)
{
    bx = blockIdx.x; by = blockIdx.y; bz = blockIdx.z;
    if (__builtin_expect(p.tail_wgs == 0, 1)) return true;
    const int own = p.gx * p.gy * p.gz;
    if (__builtin_expect(bx >= own, 0)) {
        dw_reduce_share(p.tail, bx - own, p.tail_wgs, lds);
        return false;
    }
    const int row = __builtin_amdgcn_readfirstlane(bx / p.gx);
    bx -= row * p.gx;
    bz = __builtin_amdgcn_readfirstlane(row / p.gy);
    by = row - bz * p.gy;
    return true;
}

// conv_gather.hip, conv_gather_tail.hip: the gather GEMM (conv_gather.h)
namespace gather {
constexpr int KC = 32;        // channels staged per pass
constexpr int KCS = KC + 8;   // LDS elements per patch pixel: 80 bytes, an odd number of 16-byte units
constexpr int kMaxItems = 12; // 16-byte patch items a copy thread moves per stage, at most (kernel parameter ITEMS: 6 or 12)
}
hipError_t launch_conv_gather(const GatherParams &p, int variant, hipStream_t st);
hipError_t launch_conv_gather_tail(const GatherParams &p, int variant, hipStream_t st);
// conv_tile.hip: nine-tap launches with large wave tiles (see there)
bool shape_tile(GatherParams &p, int *variant, double *cost);
hipError_t launch_tile(const GatherParams &p, int variant, hipStream_t st);
int describe_tile(const GatherParams &p, int variant, char *buf, size_t len);
// conv_dx2.hip: the 3 x 3 stride-2 data gradient, all parity classes in one launch
bool shape_dx2(const Geom &g, GatherParams &p, int *variant, double *cost);
hipError_t launch_dx2(const GatherParams &p, int variant, hipStream_t st);
int describe_dx2(const GatherParams &p, int variant, char *buf, size_t len);
// conv_wave.hip: nine-tap launches with few pixels
bool shape_wave(GatherParams &p, int *variant, double *cost);
hipError_t launch_wave(const GatherParams &p, int variant, hipStream_t st);
int describe_wave(const GatherParams &p, int variant, char *buf, size_t len);
bool shape_wave_dx2(const Geom &g, GatherParams &p, int *variant, double *cost);
hipError_t launch_wave_dx2(const GatherParams &p, int variant, hipStream_t st);
int describe_wave_dx2(const GatherParams &p, int variant, char *buf, size_t len);
// conv_pw.hip: 1 x 1 stride-1 layers
bool shape_pw(GatherParams &p, bool pool, bool record_free, int *variant, bool *gather, bool *gather_whole);
hipError_t launch_pw(const GatherParams &p, int variant, hipStream_t st);
int describe_pw(const GatherParams &p, int variant, char *buf, size_t len);

// A forward pass and a data gradient, planned; the latter with what has to be laid out ahead of it (rep).
struct FwdPlan {
    GatherParams p;
    int variant;
    size_t ws_in, ws_wt, ws_bytes; // workspace: of the channels-last input, of the repacked filter, in all
};
struct DxPlan {
    GatherParams cls[4];
    int variant[4], ncls;
    bool direct, empty_class; // dY is read where it lies; some pixels have no tap
    size_t ws_in, ws_wt, ws_bytes;
    RepackParams rep;
};
bool plan_fwd_mfma(const Geom &g, int dtype, FwdPlan *plan);
hipError_t launch_fwd_mfma(const Geom &g, FwdPlan &plan, const void *X, const void *W, const void *b, void *Y, void *Z, void *ws, hipStream_t st,
                           bool *pooled);
bool plan_dx_mfma(const Geom &g, int dtype, DxPlan *plan);
void bind_dx_mfma(DxPlan *plan, const void *W, const void *dY, void *dX, void *ws);
hipError_t launch_dx_mfma(DxPlan &plan, bool repacked, const DwReduceTail *tail, hipStream_t st);
size_t conv_mfma_workspace(const Geom &g, int dtype, bool data_grad);
// Text description of the launch shape(s) chosen; false when the geometry is not covered.
bool describe_conv_mfma(const Geom &g, int dtype, bool data_grad, char *buf, size_t len);

} // namespace cac
