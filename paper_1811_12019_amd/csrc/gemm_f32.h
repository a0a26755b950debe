// fp32 "NT" tile product on the gfx950 matrix cores: acc[128 x 128] = A[128 x K] . B[128 x K]^T with both
// operands row-major and K contiguous, v_mfma_f32_32x32x2_f32, fp32 accumulate.  Used by the panel launch of the damped
// inverse for a matrix's last, ragged block; the accumulator layout (TileAcc, acc_row, acc_col) serves every 128 x 128 tile
// product of the inverse and the preconditioner.
//
// One workgroup = 256 threads = 4 wavefronts in a 2 x 2 arrangement, each wavefront owning a 64 x 64 quadrant
// as 2 x 2 MFMA blocks (64 accumulator registers per lane).  K advances 32 at a time through LDS; the next
// K-slab is fetched into registers while the current one is multiplied.
#pragma once

#include "common.h"

namespace kfac {

constexpr int TM = 128;          // tile rows (= tile columns)
constexpr int TK = 32;           // K-slab per LDS stage
constexpr int TLD = TK + 4;      // LDS row stride in floats (keeps float4 alignment, spreads banks)
constexpr int GEMM_LDS_FLOATS = 2 * TM * TLD;          // 36,864 B; reused as epilogue staging

struct TileAcc {
    v16f c[2][2];
};

// Row / column (inside the 128 x 128 tile) of accumulator register r of MFMA block (mb, nb) for this lane.
__device__ __forceinline__ int acc_row(int wm, int mb, int r, int lane) {
    return wm * 64 + mb * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
}
__device__ __forceinline__ int acc_col(int wn, int nb, int lane) { return wn * 64 + nb * 32 + (lane & 31); }

__device__ __forceinline__ v4f load4_guard(const gfloat* p, bool row_ok, int k, int K) {
    v4f v = {0.f, 0.f, 0.f, 0.f};
    if (row_ok) {
        if (k + 3 < K) {
            v = *(const KFAC_AS1 v4f_a4*)(p + k);
        } else {
            if (k < K) v.x = p[k];
            if (k + 1 < K) v.y = p[k + 1];
            if (k + 2 < K) v.z = p[k + 2];
        }
    }
    return v;
}

// 16 rows (first, first + 8, ..) of columns k .. k + 3 of a row-major matrix at X, rows x cols elements, zero outside it.  No load
// stands under a condition (each would be waited for before the next one): rows beyond the matrix read its last one, and columns at a
// row's end are read from inside the row and moved into place.
__device__ __forceinline__ v4f tail4(v4f x, int shift) {             // elements shift .. of x, then zeros
    x = shift & 1 ? v4f{x.y, x.z, x.w, 0.f} : x;
    x = shift & 2 ? v4f{x.z, x.w, 0.f, 0.f} : x;
    return shift > 3 ? v4f{0.f, 0.f, 0.f, 0.f} : x;
}
__device__ __forceinline__ void load_rows_edge(const gfloat* X, int rows, int cols, int first, int k, v4f (&v)[16]) {
    if (cols < 4) {                                      // (uniform)
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            const int row = first + 8 * p;
            v[p] = load4_guard(X + (size_t)(row < rows ? row : 0) * cols, row < rows, k, cols);
        }
        return;
    }
    const int start = min(k, cols - 4), shift = k - start;
#pragma unroll
    for (int p = 0; p < 16; ++p) v[p] = *(const KFAC_AS1 v4f_a4*)(X + (size_t)min(first + 8 * p, rows - 1) * cols + start);
#pragma unroll
    for (int p = 0; p < 16; ++p) v[p] = tail4(v[p], first + 8 * p < rows ? shift : 4);
}

// A: first row of the tile's A operand, lda floats between rows, arows (<=128) valid rows; same for B.
__device__ __forceinline__ void tile_mma_nt(const gfloat* __restrict__ A, int lda, int arows,
                                            const gfloat* __restrict__ B, int ldb, int brows, int K,
                                            float* __restrict__ lds, TileAcc& acc) {
    constexpr int QK = TK / 4;                        // float4 per row of a slab
    constexpr int RP = 256 / QK;                      // rows per pass
    constexpr int NP = TM / RP;                       // passes per operand
    float* As = lds;
    float* Bs = lds + TM * TLD;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lr = t / QK, kq = (t % QK) * 4;         // RP rows x QK float4 per pass
    const int lm = lane & 31, h = lane >> 5;

#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc.c[mb][nb][r] = 0.f;

    v4f ra[NP], rb[NP];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int row = lr + RP * p;
            ra[p] = load4_guard(A + (size_t)row * lda, row < arows, k0 + kq, K);
            rb[p] = load4_guard(B + (size_t)row * ldb, row < brows, k0 + kq, K);
        }
    };
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += TK) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            *(v4f*)&As[(lr + RP * p) * TLD + kq] = ra[p];
            *(v4f*)&Bs[(lr + RP * p) * TLD + kq] = rb[p];
        }
        __syncthreads();
        if (k0 + TK < K) fetch(k0 + TK);
#pragma unroll
        for (int s = 0; s < TK / 8; ++s) {
            v4f a[2], b[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) a[mb] = *(const v4f*)&As[(wm * 64 + mb * 32 + lm) * TLD + 8 * s + 4 * h];
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) b[nb] = *(const v4f*)&Bs[(wn * 64 + nb * 32 + lm) * TLD + 8 * s + 4 * h];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
                        acc.c[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mb][i], b[nb][i], acc.c[mb][nb], 0, 0, 0);
        }
        __syncthreads();
    }
}

}  // namespace kfac
