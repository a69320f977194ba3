// Forward convolution and data gradient for the float path and for every geometry the MFMA kernels do not take
// (filters of more than nine taps, strides above 2): an LDS-tiled multiply-add kernel in float arithmetic, gfx950.
//
// The sum is the gather of conv_mfma.hip,
//   out[n, m, i*os + a0, j*os + b0] = bias[m] + sum_taps sum_kc W'[m][kc][tap] * in[n, kc, i*is + dh, j*is + dw],
// forward with os = 1, is = stride, (dh, dw) = (r - ph, s - pw), the data gradient with is = 1, os = stride and one
// class (a0, b0) per parity, all classes in one launch.
//
// The layers that come here are small (the single 16 -> 16 float layer of the lists is 38 MFLOP), so what bounds
// them is latency: one output per thread with its operands fetched from the caches inside the loop took 30 us
// (forward) and 19 us (data gradient) on that layer.  A workgroup of 256 threads owns 16 output channels x 64 or 256 pixels; it
// stages the input patch of CC channels (zero-padded, as floats) and the filter's part ([tap][channel][16 outputs]) in LDS, eight
// loads per thread in flight at a time, those of the next CC channels while it multiplies the present ones.  The products are the
// float matrix instruction's, 16 outputs x 16 pixels x 4 channels (float operands, products and sums; a wave has 16 or 64 of the
// pixels): two reads of LDS each, where multiply-adds took five and 16 issues, and the code a fifth of the size -- it comes through
// the instruction cache once.  Measured per call in a graph, multiply-adds / matrix instruction / filter in registers too: that layer
// 12.2 / 10.5 / 9.5 us forward and 11.4 / 8.6 / 8.1 backwards, 64 -> 64 at 13 x 13, batch 32: 31 / 21 / 18 and 34 / 20 / 16; what bounds it now is
// a pass's loads, 1.2 us for 0.5 us of products.  The error against 64 bits is the same to two digits (1.5e-7 to 4.2e-7).
// 64 pixels per workgroup when 256 would leave less than four workgroups per compute unit.
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace cac {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ uint32_t fdiv(uint32_t x, uint32_t magic) { return magic ? __umulhi(x, magic) : x; }

constexpr uint32_t kNoLoad = 0x80000000u;
// Keeps the compiler from computing what follows from `x` outside of a loop.
__device__ __forceinline__ void opaque(int &x) { asm volatile("" : "+v"(x)); }
constexpr int kTMP = 20; // floats of a filter entry in LDS: 16 outputs, padded against bank conflicts of the writes
// element at a byte offset; zero at or past the tensor's end
template <typename T> __device__ __forceinline__ float load(rsrc_t rs, uint32_t off)
{
    if constexpr (sizeof(T) == 4) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
    else return bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0));
}

struct ConvLdsParams {
    const void *in, *W, *bias;
    void *out;
    int N, M, KC, Hin, Win, Hout, Wout; // KC: input channels of the sum
    int R, S, sh, sw, ph, pw;           // of the convolution
    int C;                              // input channels of the convolution (the filter's row length)
    int Hc, Wc, ppi;                    // grid of output pixels of a class (the largest one)
    int IPT, tiles, ngrp;               // images per workgroup; tiles per image; image groups
    int PH, PWd;                        // staged patch of one image
    int cw_log2;                        // lanes of a patch row while staging, log2 (6: a whole wave, in turns)
    uint32_t m_wc, m_ppi, m_rpc, m_ph, m_rs; // division magics (m_wc, m_ppi, m_rs: 0 for 1; the others are of at least 2)
};

// T: storage type; PX: pixels per thread; DX: data gradient; CC: channels staged per pass; TAPS: 9 and 1, for float filters of 3 x 3 and
// 1 x 1 whose operands a lane reads as they lie -- the taps of its output and four channels are 36 (4) floats in a row, or four times
// 9 (1) --, else 0: the filter's part is staged in LDS.
template <typename T, int PX, bool DX, int CC, int TAPS>
__global__ void __launch_bounds__(256, (PX == 4 ? 3 : 4) - (TAPS == 9)) conv_lds_kernel(ConvLdsParams p)
{
    constexpr int TM = 16, PT = 64 * PX;
    static_assert(TAPS == 0 || (CC == 16 && sizeof(T) == 4), "");
    extern __shared__ __align__(16) float lds[];
    const int RS = TAPS ? TAPS : p.R * p.S;
    // [tap][CC][TM + 4] (TAPS: none), [CC][IPT][PH][PWd], 64 floats of nobody's
    float *sw = lds, *sx = TAPS ? lds : lds + RS * CC * kTMP;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mg = lane >> 4, l16 = lane & 15; // group of four outputs; pixel within a block of 16
    const int cls = DX ? blockIdx.z : 0, os_h = DX ? p.sh : 1, os_w = DX ? p.sw : 1, is_h = DX ? 1 : p.sh, is_w = DX ? 1 : p.sw;
    const int a0 = DX ? cls / os_w : 0, b0 = cls - a0 * os_w;
    const int grp = blockIdx.x / p.tiles, tau = blockIdx.x - grp * p.tiles;
    const int n0 = grp * p.IPT, pix0 = tau * PT, i0 = fdiv(pix0, p.m_wc), m0 = blockIdx.y * TM;
    // offsets of the taps of this class: the smallest one starts the patch (floor division, also of negatives)
    auto floor_div = [](int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); };
    const int dhmin = DX ? -floor_div(p.R - 1 - a0 - p.ph, p.sh) : -p.ph, dwmin = DX ? -floor_div(p.S - 1 - b0 - p.pw, p.sw) : -p.pw;
    const int hin0 = i0 * is_h + dhmin;

    const rsrc_t rs_in = make_rsrc(p.in, (uint32_t)p.N * p.KC * p.Hin * p.Win * (uint32_t)sizeof(T));
    const rsrc_t rs_w = make_rsrc(p.W, (uint32_t)p.M * p.KC * RS * (uint32_t)sizeof(T));
    const int rpc = p.IPT * p.PH, xplane = rpc * p.PWd, nrows = CC * rpc;
    const int woff = RS * CC * kTMP, xdump = CC * xplane + lane; // (a place of every lane's own past the patch)
    const int rpw = 64 >> p.cw_log2, cmask = (1 << p.cw_log2) - 1;
    constexpr int kRows = (DX ? CC : TM) / 4;           // rows of the filter's part per wave
    const int L = (DX ? TM : CC) * RS;                  // elements of a row
    // The patch, row by row (channel, image, patch row): one per wave and turn, or several short ones side by side, eight loads of a
    // thread to a batch, without a branch between them: what does not exist is read past the tensor (zero) and, outside the
    // row, stored past the patch.
    const int turns = (nrows + 32 * rpw - 1) / (32 * rpw), batches = turns * ((p.PWd + 63) >> 6);
    // byte offset of element (channel c0 + row's, column) of a batch
    auto offset_of = [&](int c0, int w, uint32_t rho) {
        const int c = __umulhi(rho, p.m_rpc), t = rho - c * rpc, g = __umulhi(t, p.m_ph), h = hin0 + t - g * p.PH;
        const bool ok = (w >= 0) & (w < p.Win) & (rho < (uint32_t)nrows) & (c0 + c < p.KC) & (n0 + g < p.N) & (h >= 0) & (h < p.Hin);
        return ok ? (uint32_t)((((n0 + g) * p.KC + c0 + c) * p.Hin + h) * p.Win + w) * (uint32_t)sizeof(T) : kNoLoad;
    };
    auto fetch_x = [&](int c0, int w0, int r0, float (&x)[8]) {
        opaque(r0); // (what follows from it is not to be kept in registers from pass to pass)
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = load<T>(rs_in, offset_of(c0, dwmin + w0 + (lane & cmask), r0 + 4 * q * rpw));
    };
    auto put_x = [&](int w0, int r0, const float (&x)[8]) {
        opaque(r0);
        const int col = w0 + (lane & cmask);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int rho = r0 + 4 * q * rpw;
            sx[((col < p.PWd) & (rho < nrows)) ? rho * p.PWd + col : xdump] = x[q];
        }
    };
    // The filter: rows of W [o][c][tap], their runs of (channel, tap) -- forward -- or (output, tap) -- data gradient
    // -- along the lanes; where an element of a run goes does not depend on the row.
    auto fetch_w = [&](int c0, int x0, float (&v)[2][kRows]) {
        int ln = lane;
        opaque(ln);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int xi = x0 + 64 * k + ln;
            const bool cok = (xi < L) & (xi < (DX ? (p.M - m0) * RS : (p.KC - c0) * RS));
#pragma unroll
            for (int j = 0; j < kRows; ++j) {
                const int row = wave + 4 * j, o = DX ? c0 + row : m0 + row;
                const uint32_t off = (uint32_t)((o * p.C + (DX ? m0 : c0)) * RS + xi);
                v[k][j] = load<T>(rs_w, (cok & (o < (DX ? p.KC : p.M))) ? off * (uint32_t)sizeof(T) : kNoLoad);
            }
        }
    };
    auto put_w = [&](int x0, const float (&v)[2][kRows]) {
        int ln = lane;
        opaque(ln);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int xi = x0 + 64 * k + ln, q = RS > 1 ? __umulhi(xi, p.m_rs) : xi, tap = xi - q * RS;
            const int dst = xi < L ? (DX ? tap * CC * kTMP + q : (tap * CC + q) * kTMP) : -1;
#pragma unroll
            for (int j = 0; j < kRows; ++j) {
                const int row = wave + 4 * j;
                lds[dst >= 0 ? dst + (DX ? row * kTMP : row) : xdump + woff] = v[k][j];
            }
        }
    };
    // Two batches of the patch (and two of the filter) are kept in registers, the whole of a pass on most layers; what is more is
    // fetched between two passes.  Their offsets are those of the first pass: the next one's are CC planes on.
    const int rbase = wave * rpw + (lane >> p.cw_log2);
    auto at = [&](int b, int &w0, int &r0) { // batch b: first column, this thread's first row
        const int cb = b >= turns ? b / turns : 0;
        w0 = 64 * cb;
        r0 = rbase + 32 * rpw * (b - cb * turns);
    };
    float x2[2][8], wa[2][kRows], wb[2][kRows];
    uint32_t off[2][8];
    int w1, r1; // of the second batch
    at(1, w1, r1);
    if (CC <= p.KC) // (a pass that is not full reckons for itself: 0.85 to 0.9 of the time where there is no other)
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        off[0][q] = offset_of(0, dwmin + (lane & cmask), rbase + 4 * q * rpw);
        off[1][q] = batches > 1 ? offset_of(0, dwmin + w1 + (lane & cmask), r1 + 4 * q * rpw) : kNoLoad;
    }
    constexpr int NJ = TAPS ? (DX ? 4 : 1) : 1, NF = TAPS ? 4 * TAPS / NJ : 4; // runs of a lane's floats, and their length
    float wr[NJ][NF];
    auto fetch = [&](int c0) {
        if (c0 + CC <= p.KC) {
            const uint32_t so = (uint32_t)c0 * p.Hin * p.Win * (uint32_t)sizeof(T);
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    if constexpr (sizeof(T) == 4) x2[b][q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_in, off[b][q], so, 0));
                    else x2[b][q] = bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(rs_in, off[b][q], so, 0));
                }
        } else {
            fetch_x(c0, 0, rbase, x2[0]);
            if (batches > 1) fetch_x(c0, w1, r1, x2[1]);
        }
        if constexpr (TAPS == 0) {
            fetch_w(c0, 0, wa);
            if (L > 128) fetch_w(c0, 128, wb);
        } else {
            // (a run may reach past the tensor's end: the dwords past it are zeros)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int m = m0 + l16, c = c0 + 4 * mg + j;
                const uint32_t e = (uint32_t)((DX ? c * p.C + m : m * p.C + c) * TAPS) * 4u, at = m < p.M && c < p.KC ? e : kNoLoad;
#pragma unroll
                for (int k = 0; k < NF / 4; ++k) {
                    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
                    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs_w, at, 16 * k, 0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) wr[j][4 * k + i] = __uint_as_float(v[i]);
                }
#pragma unroll
                for (int k = NF / 4 * 4; k < NF; ++k) wr[j][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_w, at, 4 * k, 0));
            }
        }
    };

    int n[PX], oi[PX], oj[PX], base[PX];
    bool ok[PX];
#pragma unroll
    for (int k = 0; k < PX; ++k) {
        const int idx = (wave * PX + k) * 16 + l16;
        int g = 0, px = pix0 + idx;
        if (p.IPT > 1) {
            g = fdiv(idx, p.m_ppi);
            px = idx - g * p.ppi;
        }
        const int i = fdiv(px, p.m_wc), j = px - i * p.Wc;
        n[k] = n0 + g;
        oi[k] = i * os_h + a0;
        oj[k] = j * os_w + b0;
        const bool in_tile = g < p.IPT && px < p.ppi; // (what the staged patch covers)
        ok[k] = in_tile && n[k] < p.N && oi[k] < p.Hout && oj[k] < p.Wout;
        base[k] = (in_tile ? (g * p.PH + (i - i0) * is_h) * p.PWd + j * is_w : 0) + mg * xplane * (TAPS ? 4 : 1); // (of this lane's channel of four)
    }
    f32x4 acc[PX];
#pragma unroll
    for (int k = 0; k < PX; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    // taps of this class: the first row and column of the filter that reach it, how far apart they are, and their offset
    const int r_0 = DX ? (a0 + p.ph) % os_h : 0, s_0 = DX ? (b0 + p.pw) % os_w : 0;
    const int row0 = ((DX ? (a0 + p.ph - r_0) / os_h : -p.ph) - dhmin) * p.PWd, col0 = (DX ? (b0 + p.pw - s_0) / os_w : -p.pw) - dwmin;
#pragma unroll 1
    for (int c0 = -CC; c0 < p.KC; c0 += CC) {
        float w[NJ][NF]; // this pass's
        if (c0 >= 0) {
            put_x(0, rbase, x2[0]);
            if (batches > 1) put_x(w1, r1, x2[1]);
            if constexpr (TAPS == 0) {
                put_w(0, wa);
                if (L > 128) put_w(128, wb);
            } else {
                // channels past the last one: whatever follows in the filter, to be multiplied with zeros, must not be infinite
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int k = 0; k < NF; ++k) w[j][k] = !DX && c0 + CC > p.KC && c0 + 4 * mg + k / TAPS >= p.KC ? 0.f : wr[j][k];
            }
#pragma unroll 1
            for (int b = 2; b < batches; ++b) {
                int w0, r0;
                at(b, w0, r0);
                fetch_x(c0, w0, r0, x2[0]);
                put_x(w0, r0, x2[0]);
            }
            if constexpr (TAPS == 0) {
#pragma unroll 1
                for (int x0 = 256; x0 < L; x0 += 128) {
                    fetch_w(c0, x0, wa);
                    put_w(x0, wa);
                }
            }
            __syncthreads();
        }
        if (c0 + CC < p.KC) fetch(c0 + CC);
        if (c0 < 0) continue;
        if constexpr (TAPS != 0) {
            constexpr int RR = TAPS == 9 ? 3 : 1;
#pragma unroll
            for (int r = 0; r < RR; ++r) {
                const int kr = DX ? (r - r_0) / (os_h == 2 ? 2 : 1) : r; // (the class's how-manieth row; strides 1 and 2)
                if (DX && (r < r_0 || (os_h == 2 && ((r - r_0) & 1)))) continue;
#pragma unroll
                for (int s = 0; s < RR; ++s) {
                    const int ksx = DX ? (s - s_0) / (os_w == 2 ? 2 : 1) : s;
                    if (DX && (s < s_0 || (os_w == 2 && ((s - s_0) & 1)))) continue;
                    const float *x = sx + row0 + col0 + (DX ? -(kr * p.PWd + ksx) : kr * p.PWd + ksx);
                    float xv[4][PX];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int k = 0; k < PX; ++k) xv[j][k] = x[j * xplane + base[k]];
                    if (PX == 4) __builtin_amdgcn_sched_barrier(0); // (not the reads of all taps ahead of the first product)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int k = 0; k < PX; ++k)
                            acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(DX ? w[j % NJ][r * RR + s] : w[0][(j * TAPS + r * RR + s) % NF], xv[j][k], acc[k], 0, 0, 0);
                }
            }
        } else {
            int xr = row0;
            for (int r = r_0; r < p.R; r += os_h, xr += DX ? -p.PWd : p.PWd) {
                const float *x = sx + xr + col0;
                const float *wt = sw + (r * p.S + s_0) * CC * kTMP + mg * kTMP + l16;
                for (int s = s_0; s < p.S; s += os_w, x += DX ? -1 : 1, wt += os_w * CC * kTMP) {
                    float wv[CC / 4], xv[CC / 4][PX];
#pragma unroll
                    for (int c = 0; c < CC / 4; ++c) {
                        wv[c] = wt[4 * c * kTMP];
#pragma unroll
                        for (int k = 0; k < PX; ++k) xv[c][k] = x[4 * c * xplane + base[k]];
                    }
#pragma unroll
                    for (int c = 0; c < CC / 4; ++c)
#pragma unroll
                        for (int k = 0; k < PX; ++k) acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[c], xv[c][k], acc[k], 0, 0, 0);
                }
            }
        }
        if (c0 + CC < p.KC) __syncthreads();
    }
    // The loop multiplied staged zeros where a tap lies outside the image: nothing as long as its weight is finite.  An
    // infinite or NaN weight has left NaN there, so a pixel with such taps that came out not finite is summed again over
    // the taps that it has, straight from memory (one pixel after the other: this code is hardly ever run, and small).
    bool again = false;
    const int dhmax = DX ? floor_div(a0 + p.ph, p.sh) : p.R - 1 - p.ph, dwmax = DX ? floor_div(b0 + p.pw, p.sw) : p.S - 1 - p.pw;
    auto row_of = [&](int k) { return DX ? (oi[k] - a0) / os_h : oi[k] * is_h; };
    auto col_of = [&](int k) { return DX ? (oj[k] - b0) / os_w : oj[k] * is_w; };
#pragma unroll
    for (int k = 0; k < PX; ++k) {
        float z = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) z = __builtin_fmaf(acc[k][e], 0.f, z);
        again |= ok[k] & (z != 0.f);
    }
    if (__any(again)) {
#pragma unroll 1
        for (int kk = 0; kk < PX; ++kk) {
            int h0 = 0, w0 = 0, img = 0;
            bool mine = false;
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < PX; ++k)
                if (k == kk) {
                    h0 = row_of(k); w0 = col_of(k); img = n[k]; mine = ok[k]; a = acc[k];
                }
            const float z = (a[0] + a[1] + a[2] + a[3]) * 0.f;
            mine &= (z != 0.f) & ((h0 + dhmin < 0) | (w0 + dwmin < 0) | (h0 + dhmax >= p.Hin) | (w0 + dwmax >= p.Win));
            if (!mine) continue;
            a = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int r = 0; r < p.R; ++r) {
                const int th = a0 + p.ph - r, dh = DX ? floor_div(th, p.sh) : r - p.ph, h = h0 + dh;
                if ((DX && th != dh * p.sh) || h < 0 || h >= p.Hin) continue;
                for (int s = 0; s < p.S; ++s) {
                    const int tw = b0 + p.pw - s, dw = DX ? floor_div(tw, p.sw) : s - p.pw, w = w0 + dw;
                    if ((DX && tw != dw * p.sw) || w < 0 || w >= p.Win) continue;
#pragma unroll 1
                    for (int c = 0; c < p.KC; ++c) {
                        const float x = load<T>(rs_in, (uint32_t)(((img * p.KC + c) * p.Hin + h) * p.Win + w) * (uint32_t)sizeof(T));
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int m = m0 + mg * 4 + e; // (past the last output: a zero)
                            const uint32_t off = (uint32_t)(((DX ? c * p.C + m : m * p.C + c) * p.R + r) * p.S + s) * (uint32_t)sizeof(T);
                            a[e] = __builtin_fmaf(x, load<T>(rs_w, m < p.M ? off : kNoLoad), a[e]);
                        }
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < PX; ++k)
                if (k == kk) acc[k] = a;
        }
    }
    T *out = (T *)p.out;
    const T *bias = (const T *)p.bias;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int m = m0 + mg * 4 + e;
        const float b = !DX && bias && m < p.M ? Elem<T>::load(bias + m) : 0.f;
#pragma unroll
        for (int k = 0; k < PX; ++k)
            if (ok[k] & (m < p.M)) Elem<T>::store(out + (((long)n[k] * p.M + m) * p.Hout + oi[k]) * p.Wout + oj[k], acc[k][e] + b);
    }
}

// A launch of the kernel: its parameters but for the tensors, pixels per thread, channels per pass, taps in registers.
struct ConvLdsPlan {
    ConvLdsParams p;
    int px, cc, taps, lds_bytes;
    double now; // see cost_lds
    dim3 grid;
};

// The launch with px pixels per thread and cc channels per pass; false when it is not possible (rows too long or a filter
// too large for LDS, tensors past 32-bit offsets).
bool shape_lds(const Geom &g, int dtype, bool dx, int px, int cc, ConvLdsPlan *plan)
{
    const long eb = dtype == CAC_F32 ? 4 : 2;
    ConvLdsParams p{};
    p.N = g.N; p.C = g.C; p.R = g.R; p.S = g.S; p.sh = g.sh; p.sw = g.sw; p.ph = g.ph; p.pw = g.pw;
    p.M = dx ? g.C : g.K; p.KC = dx ? g.K : g.C;
    p.Hin = dx ? g.P : g.H; p.Win = dx ? g.Q : g.W; p.Hout = dx ? g.H : g.P; p.Wout = dx ? g.W : g.Q;
    // (32-bit byte offsets with 2^31 reserved for what does not exist)
    if ((long)p.N * p.KC * p.Hin * p.Win * eb >= 1L << 31 || (long)p.M * p.KC * g.R * g.S * eb >= 1L << 31) return false;
    const int os_h = dx ? g.sh : 1, os_w = dx ? g.sw : 1, is_h = dx ? 1 : g.sh, is_w = dx ? 1 : g.sw;
    p.Hc = (p.Hout + os_h - 1) / os_h; p.Wc = (p.Wout + os_w - 1) / os_w;
    if ((long)p.Hc * p.Wc * p.Wc >= 1L << 32) return false; // (division by multiplication is exact below)
    p.ppi = p.Hc * p.Wc;
    const int span_h = dx ? (g.R - 1) / g.sh + 1 : g.R, span_w = dx ? (g.S - 1) / g.sw + 1 : g.S;
    const int mblocks = (p.M + 15) / 16, classes = os_h * os_w, pt = 64 * px;
    if (mblocks > 65535 || classes > 65535) return false;
    p.IPT = 2L * p.ppi <= pt ? min(pt / p.ppi, g.N) : 1;
    p.tiles = p.IPT > 1 ? 1 : (p.ppi + pt - 1) / pt;
    p.ngrp = (g.N + p.IPT - 1) / p.IPT;
    const long rows = p.IPT > 1 ? p.Hc : std::min((long)p.Hc, (long)(pt + p.Wc - 2) / p.Wc + 1);
    const long ph = std::max(2L, (rows - 1) * is_h + span_h), pw = (long)(p.Wc - 1) * is_w + span_w;
    if ((long)p.tiles * p.ngrp > 0x7fffffffL) return false;
    // Float filters of 3 x 3 and 1 x 1 are read as they lie, their taps in registers.  (Strides of 1 and 2: the kernels know the taps of a
    // parity class.  A 3 x 3 data gradient with four pixels per thread would take 256 registers and spill 59: 33.7 us against 31.3,
    // 64 -> 20 at 38 x 38, batch 20; its filter goes through LDS.)
    const bool nine = g.R == 3 && g.S == 3, known = dtype == CAC_F32 && cc == 16 && g.sh <= 2 && g.sw <= 2 && (nine || g.R * g.S == 1);
    const int taps = !known ? 0 : !nine ? 1 : dx && px == 4 ? 0 : 9;
    const long bytes = 4 * ((taps ? 0L : (long)g.R * g.S * cc * kTMP) + (long)cc * p.IPT * ph * pw + 64);
    if (bytes > 64 * 1024) return false;
    p.PH = (int)ph; p.PWd = (int)pw;
    p.cw_log2 = 0;
    while (p.cw_log2 < 6 && (1 << p.cw_log2) < p.PWd) ++p.cw_log2;
    p.m_wc = magic_of(p.Wc); p.m_ppi = magic_of(p.ppi); p.m_ph = magic_of(p.PH); p.m_rpc = magic_of(p.IPT * p.PH);
    p.m_rs = magic_of(g.R * g.S);
    plan->p = p;
    plan->px = px;
    plan->cc = cc;
    plan->taps = taps;
    plan->now = known && min(p.KC, p.M) >= 16 ? 0.62 : 1.0;
    plan->lds_bytes = (int)bytes;
    plan->grid = dim3(p.tiles * p.ngrp, mblocks, classes);
    return true;
}

// Microseconds of a launch, and of the plain kernel on the same layer: a pass costs its batches of eight loads of the
// patch, its loads of the filter and its taps x channels, once as the latency of a workgroup and once as the work of 256
// compute units; a step of the plain kernel's loop likewise, and every channel (forward) a new line of the input.  Fitted to
// 10000 random layers in each direction (1-256 channels, maps of 2-400, filters of 1-11, strides 1-3, both types): 15 %
// and 19 % rms for this kernel, 25 % and 22 % for the plain one -- when the sums were multiply-adds.  `now` is what float layers of 16
// channels and more take of that time since they are the matrix instruction's, of 1800 random ones: 3 x 3 0.6 (0.72 where the filter
// goes through LDS), 1 x 1 by the number of passes, 1.0 for one, 0.85 for two, 0.6 for many (see plan_lds).
struct LdsCost { double start, x, f, mul1, mul4, wg, wx, wf, wmul1, wmul4; };
const LdsCost kLdsCost[2] = {{0.0, 0.93, 0.0985, 0.0150, 0.0613, 0.06, 0.52, 0.0102, 0.0123, 0.0378},
                             {4.3, 1.39, 0.1067, 0.0344, 0.0851, 0.39, 0.42, 0.0543, 0.0153, 0.0380}};
struct PlainCost { double start, step, line, wstep, wg; };
const PlainCost kPlainCost[2] = {{0.5, 0.154, 0.194, 0.0715, 0.55}, {5.4, 0.125, 0.0, 0.0679, 0.41}};

double cost_lds(const Geom &g, bool dx, const ConvLdsPlan &l)
{
    const LdsCost &c = kLdsCost[dx];
    auto cdiv = [](long a, long b) { return (double)((a + b - 1) / b); };
    const int RS = g.R * g.S, rpw = 64 >> l.p.cw_log2;
    const double passes = cdiv(l.p.KC, l.cc), nx = cdiv(l.p.PWd, 64) * cdiv((long)l.cc * l.p.IPT * l.p.PH, 32 * rpw);
    const double nf = cdiv((long)(dx ? 16 : l.cc) * RS, 128) * 2 * ((dx ? l.cc : 16) / 4), mul = (double)RS / l.grid.z * l.cc;
    const double wgs = (double)l.grid.x * l.grid.y * l.grid.z;
    return c.start + l.now * hypot(passes * (c.x * nx + c.f * nf + mul * (l.px == 4 ? c.mul4 : c.mul1)),
                           wgs / 256 * (c.wg * (l.px == 4 ? 2 : 1) + passes * (c.wx * nx + c.wf * nf + mul * (l.px == 4 ? c.wmul4 : c.wmul1))));
}

double cost_plain(const Geom &g, bool dx)
{
    const PlainCost &c = kPlainCost[dx];
    // taps that some pixel has inside the image; a wave of the data gradient runs through those of all its rows
    auto valid = [](int R, int pad, int n, int out, int st) { return std::max(1.0, std::min(R - 1.0, n - 1.0 + pad) - std::max(0.0, pad - (out - 1.0) * st) + 1.0); };
    const double rows = valid(g.R, g.ph, g.H, g.P, g.sh) * (dx ? std::min(1.0, (64.0 / g.W + 1.0) / g.sh) : 1.0);
    const double steps = (dx ? g.K : g.C) * rows * valid(g.S, g.pw, g.W, g.Q, g.sw);
    const long plane = dx ? (long)g.H * g.W : (long)g.P * g.Q;
    const double wgs = (double)((plane + 255) / 256) * (((dx ? g.C : g.K) + 7) / 8) * g.N;
    return c.start + hypot(steps * c.step + (dx ? 0.0 : g.C * c.line), wgs / 256 * (steps * c.wstep + c.wg));
}

// The launch for a layer; false when it is the plain kernel's: impossible here, or slower.  Sixteen channels per pass (four
// where LDS has no room for more) and four pixels per thread once that leaves four workgroups to a compute unit, which
// hide each other's staging, are what layers of 16 channels and more want; another shape, or the plain kernel, is taken
// where it costs at least a tenth less.  That is so towards few channels, where blocks of 16 are mostly padding (call in
// us, this shape / plain kernel / as planned: 3 -> 64 3 x 3 at 32 x 32, batch 32, float, 32 / 17 / 16; data gradient of
// 64 -> 3 31 / 14 / 15; 3 -> 64 at 224 x 224, batch 2, bfloat16, data gradient 305 / 150 / 150), and for a few long rows
// (4 -> 4 at 3 x 900 21 / 11 / 11).  On 7000 random layers other than those of the fit, 31 % ran more than 5 % slower
// than on the plain kernel with this shape alone and 3 % do as planned; 16 -> 16 at 32 x 32, batch 8, 32 (plain) / 11.5.
bool plan_lds(const Geom &g, int dtype, bool dx, ConvLdsPlan *plan, double *cost_out = nullptr)
{
    const long plane = dx ? (long)((g.H + g.sh - 1) / g.sh) * ((g.W + g.sw - 1) / g.sw) : (long)g.P * g.Q;
    const long wgs4 = (plane + 255) / 256 * g.N * (((dx ? g.C : g.K) + 15) / 16) * (dx ? (long)g.sh * g.sw : 1);
    const int px0 = wgs4 >= 1024 ? 4 : 1, channels = dx ? g.K : g.C;
    // 1 x 1 layers of few channels have not gained on the plain kernel: data gradients took 1.0 to 1.4 of its time up to two passes, and
    // up to three with four pixels per thread (54 <- 20 at 14 x 32, batch 1: 6.0 against 5.2 us; 144 <- 30 at 73 x 73, batch 12: 60
    // against 44), forward passes up to two with one pixel.
    const int kept = g.R * g.S > 1 || dtype != CAC_F32 || max(g.sh, g.sw) > 2 || min(g.C, g.K) < 16 ? 0 : px0 == 1 ? 32 : dx ? 48 : 0;
    const double plain = cost_plain(g, dx) * (channels <= kept ? 0.8 : 1.0);
    double usual = 0, least = plain; // (usual: of the first possible shape with px0 pixels, 0 while there is none)
    ConvLdsPlan first{}, best{};
    for (int px : {px0, 5 - px0})
        for (int cc : {16, 4}) {
            ConvLdsPlan l;
            if (!shape_lds(g, dtype, dx, px, cc, &l)) continue;
            const double cost = cost_lds(g, dx, l);
            if (px == px0 && usual == 0) { usual = cost; first = l; }
            if (cost < least) { least = cost; best = l; }
            if (channels > 8) break; // (passes of four only where those of sixteen do not fit: the same work in more passes)
        }
    const double otherwise = usual > 0 ? usual : plain;
    if (cost_out) *cost_out = least < 0.9 * otherwise ? least : otherwise;
    if (least < 0.9 * otherwise) *plan = best;
    else if (usual > 0) *plan = first;
    else return false;
    return plan->px != 0;
}

template <typename T, bool DX> hipError_t launch(const ConvLdsPlan &l, hipStream_t st)
{
#define CAC_LDS(PX, CC, TAPS) hipLaunchKernelGGL((conv_lds_kernel<T, PX, DX, CC, TAPS>), l.grid, dim3(256), l.lds_bytes, st, l.p)
    if constexpr (sizeof(T) == 4) {
        if (l.taps) {
            if (l.taps == 9) {
                if (l.px == 1) CAC_LDS(1, 16, 9);
                else if constexpr (!DX) CAC_LDS(4, 16, 9);
            } else {
                if (l.px == 4) CAC_LDS(4, 16, 1); else CAC_LDS(1, 16, 1);
            }
            return hipGetLastError();
        }
    }
    if (l.cc == 16) {
        if (l.px == 4) CAC_LDS(4, 16, 0); else CAC_LDS(1, 16, 0);
    } else {
        if (l.px == 4) CAC_LDS(4, 4, 0); else CAC_LDS(1, 4, 0);
    }
#undef CAC_LDS
    return hipGetLastError();
}

} // namespace

double cost_without_mfma(const Geom &g, int dtype, bool dx)
{
    ConvLdsPlan l;
    double cost;
    plan_lds(g, dtype, dx, &l, &cost);
    return cost;
}

bool launch_fwd_lds(const Geom &g, int dtype, const void *X, const void *W, const void *b, void *Y, hipStream_t st, hipError_t *err)
{
    ConvLdsPlan l;
    if (!plan_lds(g, dtype, false, &l)) return false;
    l.p.in = X; l.p.W = W; l.p.bias = b; l.p.out = Y;
    *err = dtype == CAC_F32 ? launch<float, false>(l, st) : launch<bf16_t, false>(l, st);
    return true;
}

bool launch_dx_lds(const Geom &g, int dtype, const void *W, const void *dY, void *dX, hipStream_t st, hipError_t *err)
{
    ConvLdsPlan l;
    if (!plan_lds(g, dtype, true, &l)) return false;
    l.p.in = dY; l.p.W = W; l.p.bias = nullptr; l.p.out = dX;
    *err = dtype == CAC_F32 ? launch<float, true>(l, st) : launch<bf16_t, true>(l, st);
    return true;
}

bool describe_lds(const Geom &g, int dtype, bool data_grad, char *buf, size_t len)
{
    ConvLdsPlan l;
    if (!plan_lds(g, dtype, data_grad, &l)) return false;
    snprintf(buf, len, "conv_lds tile=16ch x %dpx (%d per thread) ch/pass=%d img/tile=%d patch=%dx%d grid=%ux%ux%u lds=%dB", 64 * l.px, l.px, l.cc, l.p.IPT,
             l.p.PH, l.p.PWd, l.grid.x, l.grid.y, l.grid.z, l.lds_bytes);
    return true;
}

} // namespace cac
