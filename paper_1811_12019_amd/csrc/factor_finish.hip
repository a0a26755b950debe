// Second pass of the factor builds: partial sums added up, scaled, and written as plain square, running average or packed triangle.
#include "factor_batch.h"

namespace kfac {

// Second pass of split matrix-core builds: the per-split partial tiles summed in a fixed order, scaled, written with
// their mirror, and the bias row from the column sums (one workgroup per 256 columns).  One workgroup per 32 x 32 sub-block of a
// tile (partial reads are 128-byte runs, the mirror goes through an LDS transpose), or, for narrow matrices of many rows (few
// sub-blocks, hundreds of splits), per 8 x 32 of it, the four wavefronts sharing out the splits.
constexpr int RD_MANY_SUMS = 8 * 33 + 8, RD_MANY_FLOATS = RD_MANY_SUMS + 3 * 64 * 4;
static_assert(RD_MANY_SUMS % 4 == 0 && 32 * 33 <= SH_BLOCK_FLOATS, "LDS of reduce_partials");

template <int GROUPS>
__device__ __forceinline__ v4f sum_partials(const gfloat* src, size_t stride, int nsplit, int grp) {
    v4f s = {0.f, 0.f, 0.f, 0.f};
    int sp = grp;
    for (; sp + 7 * GROUPS < nsplit; sp += 8 * GROUPS) {
        v4f p[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) p[k] = *(const KFAC_AS1 v4f*)(src + (size_t)(sp + k * GROUPS) * stride);
#pragma unroll
        for (int k = 0; k < 8; ++k) s += p[k];
    }
    for (; sp < nsplit; sp += GROUPS) s += *(const KFAC_AS1 v4f*)(src + (size_t)sp * stride);
    return s;
}

__device__ __forceinline__ void reduce_bias(const View& v, const FactorPlan& pl, const Partial& part, const OutSpec& os, float scale, int c) {
    const int d = v.dout;
    if (c == 0) emit_sym(os, d, d - 1, d - 1, (float)v.u.R * scale, false);
    const int co = result_index(v, c);
    if (co < 0) return;
    const size_t stride = (size_t)pl.tiles_dim * pl.tw;
    float s = 0.f;
#pragma unroll 8
    for (int sp = 0; sp < pl.nsplit; ++sp) s += part.sums[sp * stride + c];
    emit_sym(os, d, d - 1, co, s * scale, true);
}

template <int GROUPS>
__device__ __forceinline__ void reduce_partials(const View& v, const FactorPlan& pl, const Partial& part, const OutSpec& os, float scale,
                                                int local, float* lds) {
    const int t = threadIdx.x;
    const int D = v.u.d, d = v.dout, T = pl.tw, SB = T / 32, subs = SB * SB;
    constexpr bool many = GROUPS > 1;
    const int wgs = pl.ntiles * subs * (many ? 4 : 1);
    if (local >= wgs) return reduce_bias(v, pl, part, os, scale, (local - wgs) * 256 + t);
    const int eighth = many ? local & 3 : 0;                         // which 8 rows of the sub-block
    if (many) local >>= 2;
    const int tile = local / subs, sub = local - tile * subs;
    int I, J;
    tri_decode_blocked<4>(pl.tiles_dim, tile, I, J);                 // (the tile kernel's order)
    const int si = sub / SB, sj = sub - si * SB;
    const int row0 = I * T + si * 32, col0 = J * T + sj * 32;
    if (row0 < col0 || row0 >= D || col0 >= D) return;               // above the diagonal, or outside the matrix
    const bool dg = row0 == col0, packed = os.mode == OUT_PACKED;
    const gfloat* src = part.tiles + (size_t)tile * pl.tile_floats + (pl.ntiles == 1 ? si * (si + 1) / 2 + sj : si * SB + sj) * 1024;
    const size_t stride = (size_t)pl.ntiles * pl.tile_floats;
    gfloat* __restrict__ out = os.dst;
    float (*tr)[33] = (float (*)[33])lds;
    if constexpr (many) {
        static_assert(GROUPS == 4, "one group per wavefront");
        const int grp = t >> 6, lane = t & 63;
        v4f s = sum_partials<GROUPS>(src + eighth * 256 + lane * 4, stride, pl.nsplit, grp);
        v4f* gsum = (v4f*)(lds + RD_MANY_SUMS);                        // the groups' sums, in a fixed order
        if (grp > 0) gsum[(grp - 1) * 64 + lane] = s;
        __syncthreads();
        if (grp == 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) s += gsum[k * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) tr[4 * (lane >> 5) + i][lane & 31] = s[i] * scale;
        }
        __syncthreads();
        {
            const int lr = t >> 5, lc = t & 31, row = row0 + eighth * 8 + lr, col = col0 + lc;
            const int ro = result_index(v, row), co = result_index(v, col);
            if (!packed && ro >= 0 && co >= 0 && !(dg && row < col)) {
                float val = tr[lr][lc];
                if (os.mode == OUT_EMA) tr[lr][lc] = val = fmaf(os.decay, out[(size_t)ro * d + co], os.one_minus * val);
                out[(size_t)ro * d + co] = val;
            }
        }
        __syncthreads();
        const int lr = t & 7, lc = t >> 3, row = row0 + eighth * 8 + lr, col = col0 + lc;
        const int ro = result_index(v, row), co = result_index(v, col);
        if (ro < 0 || co < 0 || (dg && (packed ? row < col : row <= col))) return;
        out[packed ? packed_row_base(min(ro, co), d) + max(ro, co) : (size_t)co * d + ro] = tr[lr][lc];
        return;
    }
    v4f s = sum_partials<1>(src + t * 4, stride, pl.nsplit, 0);
    // from the registers' order (Partial) to four columns of one row per thread
    {
        const int q = t >> 6, lane = t & 63;
#pragma unroll
        for (int i = 0; i < 4; ++i) tr[8 * q + 4 * (lane >> 5) + i][lane & 31] = s[i];
    }
    __syncthreads();
    const int lr = t >> 3, lc = (t & 7) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = tr[lr][lc + i];
    __syncthreads();
    s *= scale;
    {
        const int row = row0 + lr, ro = result_index(v, row);
        int co[4];
        bool ok[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            co[q] = result_index(v, col0 + lc + q);
            ok[q] = ro >= 0 && co[q] >= 0 && !(dg && row < col0 + lc + q);
        }
        if (os.mode == OUT_EMA) {
            float old[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) old[q] = ok[q] ? out[(size_t)ro * d + co[q]] : 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] = fmaf(os.decay, old[q], os.one_minus * s[q]);
        }
        if (!packed) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (ok[q]) out[(size_t)ro * d + co[q]] = s[q];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) tr[lr][lc + q] = s[q];
    __syncthreads();
    // transposed: thread (lr, lc .. lc + 3) holds column col0 + lr of rows row0 + lc ..
    const int col = col0 + lr, co = result_index(v, col);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = row0 + lc + q, ro = result_index(v, row);
        if (ro < 0 || co < 0 || (dg && (packed ? row < col : row <= col))) continue;
        if (packed) out[packed_row_base(min(ro, co), d) + max(ro, co)] = tr[lc + q][lr];
        else out[(size_t)co * d + ro] = tr[lc + q][lr];
    }
}

// The second pass of a call's builds.  GROUPS 1: few row ranges, and factors from the parts that their tap pairs share; 4: many
// ranges.
template <int GROUPS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void factor_tile_reduce_kernel(FBatch b) {
    __shared__ __attribute__((aligned(16))) float lds[GROUPS == 1 ? SH_BLOCK_FLOATS : RD_MANY_FLOATS];
    int local;
    const int m = fbatch_locate(b, blockIdx.x, local);
    kfac_factor_item it;
    Unfold u;
    View v;
    fbatch_item(b, m, it, u, v);
    const float scale = it.scale == 0.f ? 1.0f / (float)u.R : it.scale;
    if constexpr (GROUPS == 1) {
        if (v.shared) {
            assemble_blocks(v, plan_shared(v, b.share[m]), shared_ws(v, it.ws), out_spec(it), scale, local, lds);
            return;
        }
    }
    const FactorPlan pl = plan_tiles(v, b.share[m]);
    reduce_partials<GROUPS>(v, pl, partial_of(v, pl, it.ws), out_spec(it), scale, local, lds);
}

// The same for shared parts in (channel, tap) order.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void factor_channels_kernel(FBatch b) {
    __shared__ __attribute__((aligned(16))) float lds[SH_CHANNEL_FLOATS];
    int local;
    const int m = fbatch_locate(b, blockIdx.x, local);
    kfac_factor_item it;
    Unfold u;
    View v;
    fbatch_item(b, m, it, u, v);
    const float scale = it.scale == 0.f ? 1.0f / (float)u.R : it.scale;
    assemble_channels(v, plan_shared(v, b.share[m]), shared_ws(v, it.ws), out_spec(it), scale, local, lds);
}

int launch_factor_finish(const FBatch& b, int list, hipStream_t stream) {
    if (b.count == 0) return KFAC_OK;
    const dim3 grid(b.prefix[b.count]);
    if (list == FINISH_FEW) KFAC_LAUNCH(factor_tile_reduce_kernel<1>, grid, dim3(256), stream, b);
    else if (list == FINISH_MANY) KFAC_LAUNCH(factor_tile_reduce_kernel<4>, grid, dim3(256), stream, b);
    else KFAC_LAUNCH(factor_channels_kernel, grid, dim3(256), stream, b);
    return KFAC_OK;
}

}  // namespace kfac
