// Repacking of a tensor that the matrix-core factor builder cannot read as it lies: NCHW -> channels last, and channel
// counts that are no multiple of a 16-byte vector -> padded with zero channels.  One read and one write of the tensor
// (HBM bound), against a gather of every tap of every element by every tile.
// Workgroup = 64 pixels x 64 channels of one image, transposed through LDS: loads run along pixels, stores along channels.
#pragma once

#include "factor_tile.h"

namespace kfac {

constexpr int RP_T = 64;
constexpr int RP_LDS_BYTES = RP_T * (RP_T + 1) * 4;

static inline __host__ __device__ int repack_wgs(const Unfold& u, const View& v) {     // u: the caller's tensor
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
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int e = 0; e < RP_T * VPR / 256; ++e) {
        const int p = (t + 256 * e) / VPR, q = (t + 256 * e) % VPR;
        const unsigned* s = td + p * (LDE / EPD) + 4 * q;
        const v4u o = {s[0], s[1], s[2], s[3]};
        if (p0 + p < hw && c0 + q * 4 * EPD < Cp)
            *(KFAC_AS1 v4u*)(dst + (((size_t)n * hw + p0 + p) * Cp + c0) / EPD + 4 * q) = o;
    }
}

}  // namespace kfac
