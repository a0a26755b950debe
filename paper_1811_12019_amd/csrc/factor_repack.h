// Repacking of a tensor that the matrix-core factor builder cannot read as it lies: NCHW -> channels last, and channel
// counts that are no multiple of a 16-byte vector -> padded with zero channels.  One read and one write of the tensor
// (HBM bound), against a gather of every tap of every element by every tile.  All tensors of ResNet-50 from NCHW took, in bf16 at
// batch 32 (2.8 GB moved), 587 us = 4.7 TB/s, in fp32 at batch 8 276 us = 5.0 TB/s; most are read as they lie now (reads_planes).
// Workgroup = 64 pixels x 64 channels of one image, transposed through LDS: loads run along pixels, stores along channels.
#pragma once

#include "factor_tile.h"

namespace kfac {

constexpr int RP_T = 64;
constexpr int RP_LDS_BYTES = RP_T * (RP_T + 1) * 4;

static inline __host__ __device__ int repack_wgs(const Unfold& u, const View& v) {     // u: the caller's tensor
    if (v.rows) return ceil_div(v.u.N * v.u.H * (v.u.W / 2), 256);
    return u.N * ceil_div(u.H * u.W, RP_T) * ceil_div(v.u.C, RP_T);
}
static inline __host__ __device__ size_t repack_bytes(const View& v) {
    const size_t b = (size_t)v.u.N * v.u.H * v.u.W * v.u.C * (v.u.dtype == KFAC_F32 ? 4 : 2);
    return v.repack ? (b + 255) / 256 * 256 : 0;
}

template <typename E>
__device__ __forceinline__ void repack_tile(const Unfold& u, const View& v, const KFAC_AS1 E* __restrict__ x,
                                            KFAC_AS1 unsigned* __restrict__ dst, int wg, unsigned char* smem) {
    constexpr int LDE = sizeof(E) == 4 ? RP_T + 1 : RP_T + 2;       // tile row stride in elements: an odd number of dwords
    constexpr int EPD = 4 / sizeof(E);                              // elements per dword
    E* tile = (E*)smem;
    const int hw = u.H * u.W, Cp = v.u.C;
    const int nc = ceil_div(Cp, RP_T), np = ceil_div(hw, RP_T);
    const int cb = wg % nc, rest = wg / nc, pb = rest % np, n = rest / np;
    const int c0 = cb * RP_T, p0 = pb * RP_T;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    E val[16];
    if (u.layout == KFAC_NCHW) {
        const bool pok = p0 + lane < hw;
        const KFAC_AS1 E* src = x + ((size_t)n * u.C + c0) * hw + (pok ? p0 + lane : 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {                              // (clamped, not guarded: all loads go out together)
            const int c = wave + 4 * i;
            val[i] = src[(size_t)min(c, u.C - 1 - c0) * hw];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int c = wave + 4 * i;
            tile[lane * LDE + c] = pok && c0 + c < u.C ? val[i] : (E)0;
        }
    } else {
        const bool cok = c0 + lane < u.C;
        const KFAC_AS1 E* src = x + ((size_t)n * hw + p0) * u.C + (cok ? c0 + lane : 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) val[i] = src[(size_t)min(wave + 4 * i, hw - 1 - p0) * u.C];
#pragma unroll
        for (int i = 0; i < 16; ++i) tile[(wave + 4 * i) * LDE + lane] = cok ? val[i] : (E)0;
    }
    __syncthreads();
    constexpr int VPR = RP_T / (4 * EPD);                           // 16-byte vectors per pixel of the tile
    const unsigned* td = (const unsigned*)smem;
#pragma unroll
    for (int e = 0; e < RP_T * VPR / 256; ++e) {
        const int p = (t + 256 * e) / VPR, q = (t + 256 * e) % VPR;
        const unsigned* s = td + p * (LDE / EPD) + 4 * q;
        const v4u o = {s[0], s[1], s[2], s[3]};
        if (p0 + p < hw && c0 + q * 4 * EPD < Cp)
            *(KFAC_AS1 v4u*)(dst + (((size_t)n * hw + p0 + p) * Cp + c0) / EPD + 4 * q) = o;
    }
}

// View::rows: the image with its zero padding, four channels to a pixel; one thread per pair of pixels (16 bytes).
__device__ __forceinline__ void repack_rows(const Unfold& u, const View& v, const KFAC_AS1 unsigned short* __restrict__ x,
                                            KFAC_AS1 unsigned* __restrict__ dst, int wg) {
    const int W2 = v.u.W / 2;
    const int id = wg * 256 + (int)threadIdx.x;
    if (id >= v.u.N * v.u.H * W2) return;
    const int row = id / W2, x2 = id - row * W2, n = row / v.u.H, y = row - n * v.u.H - u.pad;
    const size_t cs = u.layout == KFAC_NHWC ? 1 : (size_t)u.H * u.W, ps = u.layout == KFAC_NHWC ? u.C : 1;
    unsigned val[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {                                   // (element 0 stands in for the padding: no branches)
        const int xx = 2 * x2 + (e >> 2) - u.pad, c = e & 3;
        const bool ok = (unsigned)y < (unsigned)u.H && (unsigned)xx < (unsigned)u.W && c < u.C;
        const size_t at = (size_t)n * u.C * u.H * u.W + ((size_t)y * u.W + xx) * ps + c * cs;
        val[e] = ok ? 1u : 0u;
        val[e] *= x[ok ? at : 0];
    }
    const v4u o = {val[0] | val[1] << 16, val[2] | val[3] << 16, val[4] | val[5] << 16, val[6] | val[7] << 16};
    *(KFAC_AS1 v4u*)(dst + (size_t)id * 4) = o;
}

}  // namespace kfac
