// Kronecker-factor builders: A = scale * Xbar^T Xbar and G = scale * Gamma^T Gamma (Sec. 3.2, Eq. 5;
// Algorithm 1 stages 1 and 2) computed straight from the activation / output-gradient tensor.  The
// unfolded patch matrix is never materialised: tiles of it are gathered on the fly into LDS.
//
// Kernels:
//   factor_tile_kernel     matrix cores, channels-last tensors of any dtype, and NCHW ones whose rows are their pixels, as they lie
//                          (factor_tile.h); many builds share one launch
//                          (workgroup -> (build, tile) through a prefix table).
//   factor_repack_kernel   brings tensors in other layouts, or with channel counts that are no multiple of a 16-byte
//                          vector, into that form first (factor_repack.h).
//   factor_generic_kernel  small builds that would have to be repacked, and whatever the others cannot take (tensors at
//                          odd addresses, 32,768 columns), fp32 FMA.
// All enumerate only the lower-triangular tiles of the symmetric output and mirror them, and all can split the R unfolded
// rows over several workgroups (deterministic two-pass reduction through the caller's workspace, no float atomics).
#include <algorithm>

#include "common.h"
#include "factor_batch.h"
#include "factor_cut.h"

namespace kfac {

// Column of the unfolded matrix -> (channel, tap row, tap column); kind: 0 data, 1 bias (constant 1), 2 padding (0)
struct ColInfo {
    int c, i, j, kind;
};

__device__ __forceinline__ ColInfo decode_col(const Unfold& u, int col) {
    ColInfo ci;
    ci.c = ci.i = ci.j = 0;
    if (col >= u.d) {
        ci.kind = 2;
    } else if (u.has_bias && col == u.d - 1) {
        ci.kind = 1;
    } else {
        ci.kind = 0;
        if (u.order == KFAC_ORDER_C_KH_KW) {
            int khw = u.kh * u.kw;
            ci.c = col / khw;
            int rem = col - ci.c * khw;
            ci.i = rem / u.kw;
            ci.j = rem - ci.i * u.kw;
        } else {
            int tap = col / u.C;
            ci.c = col - tap * u.C;
            ci.i = tap / u.kw;
            ci.j = tap - ci.i * u.kw;
        }
    }
    return ci;
}

__device__ __forceinline__ void generic_tile(const Unfold& u, const KFAC_AS1 void* __restrict__ x, float scale, const OutSpec& os,
                                             gfloat* __restrict__ partial, int rows_per_split, int tile, int ntiles, int split, int nsplit) {
    __shared__ float As[GK][GT + 4];
    __shared__ float Bs[GK][GT + 4];
    __shared__ int rowN[2][GK], rowY[2][GK], rowX[2][GK];

    const int t = threadIdx.x;
    int I, J;
    tri_decode(tile, I, J);
    const int r_begin = split * rows_per_split;
    const int r_end = min(u.R, r_begin + rows_per_split);

    const int m = t & 63, kb = t >> 6;
    const ColInfo ca = decode_col(u, I * GT + m);
    const ColInfo cb = decode_col(u, J * GT + m);
    const int tx = t & 15, ty = t >> 4;

    // A slab's rows are located, and its elements fetched, while the slab before is multiplied.  Elements are read without conditions
    // (what is not there from the tensor's first element) and chosen afterwards: a load under a condition is waited for before the
    // next one goes out, eight trips to memory a slab (512 rows of 145 columns 15.2 -> 12.5 us).
    auto locate_rows = [&](int r0, int buf) {
        if (t < GK) {
            const int r = min(r0 + t, u.R - 1);
            const int n = r / (u.Ho * u.Wo), rem = r - n * (u.Ho * u.Wo), yo = rem / u.Wo, xo = rem - yo * u.Wo;
            rowN[buf][t] = r0 + t < r_end ? n : -1;
            rowY[buf][t] = yo * u.stride - u.pad;
            rowX[buf][t] = xo * u.stride - u.pad;
        }
    };
    float va[4], vb[4];
    auto fetch = [&](int buf) {
        int ia[4], ib[4];                                        // element, or -1: 0, -2: 1 (bias column)
        auto index_of = [&](const ColInfo& c, int n, int y0, int x0) -> int {
            const int y = y0 + c.i, xx = x0 + c.j;
            const bool in = (n >= 0) & ((unsigned)y < (unsigned)u.H) & ((unsigned)xx < (unsigned)u.W);
            const int idx = u.layout == KFAC_NHWC ? ((n * u.H + y) * u.W + xx) * u.C + c.c : ((n * u.C + c.c) * u.H + y) * u.W + xx;
            return c.kind == 1 ? (n >= 0 ? -2 : -1) : c.kind == 0 && in ? idx : -1;
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = kb + 4 * e, n = rowN[buf][k], y0 = rowY[buf][k], x0 = rowX[buf][k];
            ia[e] = index_of(ca, n, y0, x0);
            ib[e] = index_of(cb, n, y0, x0);
        }
        if (u.dtype == KFAC_F32) {                               // (uniform)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                va[e] = ((const gfloat*)x)[max(ia[e], 0)];
                vb[e] = ((const gfloat*)x)[max(ib[e], 0)];
            }
        } else {
            uint16_t ha[4], hb[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ha[e] = ((const KFAC_AS1 uint16_t*)x)[max(ia[e], 0)];
                hb[e] = ((const KFAC_AS1 uint16_t*)x)[max(ib[e], 0)];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                va[e] = u.dtype == KFAC_BF16 ? bf16_bits_to_float(ha[e]) : half_bits_to_float(ha[e]);
                vb[e] = u.dtype == KFAC_BF16 ? bf16_bits_to_float(hb[e]) : half_bits_to_float(hb[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            va[e] = ia[e] >= 0 ? va[e] : ia[e] == -2 ? 1.f : 0.f;
            vb[e] = ib[e] >= 0 ? vb[e] : ib[e] == -2 ? 1.f : 0.f;
        }
    };
    locate_rows(r_begin, 0);
    __syncthreads();
    fetch(0);
    float acc[4][4] = {};
    int buf = 0;
    for (int r0 = r_begin; r0 < r_end; r0 += GK) {
        buf ^= 1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            As[kb + 4 * e][m] = va[e];
            Bs[kb + 4 * e][m] = vb[e];
        }
        locate_rows(r0 + GK, buf);
        __syncthreads();
        fetch(buf);                                              // (behind the last slab: nothing is there)
#pragma unroll
        for (int k = 0; k < GK; ++k) {
            float a[4], b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a[q] = As[k][ty * 4 + q];
                b[q] = Bs[k][tx * 4 + q];
            }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[p][q] = fmaf(a[p], b[q], acc[p][q]);
        }
        __syncthreads();
    }

    if (nsplit == 1) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int row = I * GT + ty * 4 + p, col = J * GT + tx * 4 + q;
                if (row < u.d && col < u.d) emit_sym(os, u.d, row, col, acc[p][q] * scale, I != J);
            }
    } else {
        gfloat* dst = partial + ((size_t)split * ntiles + tile) * (GT * GT);
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) dst[(ty * 4 + p) * GT + tx * 4 + q] = acc[p][q];
    }
}

// Second pass of a split build: sum the per-split partial tiles in a fixed order, scale, write the tile and its
// mirror.  One workgroup per 32 x 32 sub-block of a tile: every thread owns four consecutive columns of one row, so
// partial reads are 128-byte runs; the mirror goes through an LDS transpose.
template <int T>
__device__ __forceinline__ void factor_reduce_block(const gfloat* __restrict__ partial, int nsplit, int ntiles,
                                                    int tile, int sub, int d, float scale, const OutSpec& os,
                                                    float (*tr)[33]) {
    int I, J;
    tri_decode(tile, I, J);
    constexpr int SB = T / 32;
    const int si = sub / SB, sj = sub - si * SB;
    const int lr = threadIdx.x >> 3, lc = (threadIdx.x & 7) * 4;
    const int trow = si * 32 + lr, tcol = sj * 32 + lc;              // inside the tile
    const int row = I * T + trow, col = J * T + tcol;
    if (I * T + si * 32 >= d || J * T + sj * 32 >= d) return;       // whole sub-block outside the matrix
    v4f s = {0.f, 0.f, 0.f, 0.f};
    if (row < d && col < d) {
        const gfloat* src = partial + (size_t)tile * (T * T) + trow * T + tcol;
        const size_t stride = (size_t)ntiles * (T * T);
        auto at = [&](int sp) { return *(const KFAC_AS1 v4f*)(src + (size_t)sp * stride); };
        int sp = 0;
        for (; sp + 8 <= nsplit; sp += 8) {
            const v4f a = at(sp), b = at(sp + 1), c = at(sp + 2), e = at(sp + 3), f = at(sp + 4), g = at(sp + 5), h = at(sp + 6), k = at(sp + 7);
            s += ((a + b) + (c + e)) + ((f + g) + (h + k));
        }
        if (sp + 4 <= nsplit) {
            const v4f a = at(sp), b = at(sp + 1), c = at(sp + 2), e = at(sp + 3);
            s += (a + b) + (c + e);
            sp += 4;
        }
        for (; sp < nsplit; ++sp) s += at(sp);
        s *= scale;
        gfloat* __restrict__ out = os.dst;
        if (os.mode == OUT_PACKED) {                                 // only elements on or above the diagonal exist
            if (I == J) {
                const size_t rb = packed_row_base(row, d);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (col + q < d && col + q >= row) out[rb + col + q] = s[q];
            }
        } else {
            if (os.mode == OUT_EMA) {
                if (col + 3 < d) {
                    const v4f o = *(const KFAC_AS1 v4f_a4*)(out + (size_t)row * d + col);
#pragma unroll
                    for (int q = 0; q < 4; ++q) s[q] = fmaf(os.decay, o[q], os.one_minus * s[q]);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (col + q < d) s[q] = fmaf(os.decay, out[(size_t)row * d + col + q], os.one_minus * s[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (col + q < d) out[(size_t)row * d + col + q] = s[q];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) tr[lr][lc + q] = s[q];
    if (I == J) return;                                              // uniform: diagonal tiles hold their own mirror
    __syncthreads();
    // transposed: thread (lr, lc..lc+3) now owns mirrored row (J*T + sj*32 + lr), columns I*T + si*32 + lc..+3
    const int mrow = J * T + sj * 32 + lr, mcol = I * T + si * 32 + lc;
    if (mrow < d) {
        gfloat* __restrict__ mout = os.dst + (os.mode == OUT_PACKED ? packed_row_base(mrow, d) : (size_t)mrow * d);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (mcol + q < d) mout[mcol + q] = tr[lc + q][lr];
    }
}

// One build (its plan worked out by the host), and the builds of a call in one launch (one by one, two launches each, they would follow
// each other's ends: eight builds of 512 rows of 145 columns 88.8 us, now 20.4; fifteen of 75 rows of 71 columns 155.6, now 14.0).
__global__ __launch_bounds__(256) void factor_generic_kernel(Unfold u, const void* x, float scale, OutSpec os, float* partial,
                                                             int rows_per_split) {
    generic_tile(u, (const KFAC_AS1 void*)x, scale, os, as_global(partial), rows_per_split, blockIdx.x, gridDim.x, blockIdx.y, gridDim.y);
}

constexpr int GENERIC_SUBS = (GT / 32) * (GT / 32);          // workgroups of the second pass to a tile
__global__ __launch_bounds__(256) void factor_reduce_kernel(const float* partial, int nsplit, int d, float scale, OutSpec os) {
    __shared__ float tr[32][33];
    factor_reduce_block<GT>(as_global(partial), nsplit, gridDim.x, blockIdx.x, blockIdx.y, d, scale, os, tr);
}

__device__ __forceinline__ void generic_item(const FBatch& b, int m, kfac_factor_item& it, Unfold& u, FactorPlan& p, float& scale) {
    it = uniform(b.table[b.index[m]]);
    if (it.op == KFAC_OP_FACTOR_A) make_unfold_A(&it.desc, &u); else make_unfold_G(&it.desc, &u);
    p = plan_generic(u);
    scale = it.scale == 0.f ? 1.0f / (float)u.R : it.scale;
}
__global__ __launch_bounds__(256) void factor_generic_batch_kernel(FBatch b) {
    int local;
    const int m = fbatch_locate(b, blockIdx.x, local);
    kfac_factor_item it;
    Unfold u;
    FactorPlan p;
    float scale;
    generic_item(b, m, it, u, p, scale);
    const int split = local / p.ntiles;
    generic_tile(u, (const KFAC_AS1 void*)it.x, scale, out_spec(it), (gfloat*)it.ws, p.rows_per_split, local - split * p.ntiles, p.ntiles,
                 split, p.nsplit);
}
__global__ __launch_bounds__(256) void factor_reduce_batch_kernel(FBatch b) {
    __shared__ float tr[32][33];
    int local;
    const int m = fbatch_locate(b, blockIdx.x, local);
    kfac_factor_item it;
    Unfold u;
    FactorPlan p;
    float scale;
    generic_item(b, m, it, u, p, scale);
    factor_reduce_block<GT>((const gfloat*)it.ws, p.nsplit, p.ntiles, local / GENERIC_SUBS, local % GENERIC_SUBS, u.d, scale, out_spec(it), tr);
}

__global__ __launch_bounds__(256) void factor_repack_kernel(FBatch b) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[RP_LDS_BYTES];
    int local;
    const int m = fbatch_locate(b, blockIdx.x, local);
    kfac_factor_item it;
    Unfold u;
    View v;
    fbatch_item<false>(b, m, it, u, v);
    if (v.rows) repack_rows(u, v, (const KFAC_AS1 unsigned short*)it.x, (KFAC_AS1 unsigned*)it.ws, local);
    else if (u.dtype == KFAC_F32) repack_tile<float>(u, v, (const gfloat*)it.x, (KFAC_AS1 unsigned*)it.ws, local, smem);
    else repack_tile<unsigned short>(u, v, (const KFAC_AS1 unsigned short*)it.x, (KFAC_AS1 unsigned*)it.ws, local, smem);
}

static int check_item(const kfac_factor_item& it, Unfold* u) {
    if (!item_unfold(it, u)) return KFAC_ERR_INVALID_ARG;
    if (!it.x) return KFAC_ERR_INVALID_ARG;
    // exactly one destination: the fresh factor (square or packed) or the running average it is folded into
    if (it.running ? (it.out != nullptr || it.packed != 0 || !(it.decay >= 0.f && it.decay <= 1.f)) : !it.out) return KFAC_ERR_INVALID_ARG;
    if (it.packed != 0 && it.packed != 1) return KFAC_ERR_INVALID_ARG;
    const size_t need = item_ws_bytes(*u);
    if (need > 0 && (!it.ws || ((uintptr_t)it.ws & 255) || it.ws_bytes < need)) return KFAC_ERR_WORKSPACE;
    return KFAC_OK;
}

static int run_generic(const Unfold& u, const kfac_factor_item& it, hipStream_t stream) {
    const float scale = it.scale == 0.f ? 1.0f / (float)u.R : it.scale;
    FactorPlan p = plan_generic(u);
    dim3 grid(p.ntiles, p.nsplit);
    KFAC_LAUNCH(factor_generic_kernel, grid, dim3(256), stream, u, it.x, scale, out_spec(it), (float*)it.ws, p.rows_per_split);
    if (p.nsplit > 1)
        KFAC_LAUNCH(factor_reduce_kernel, dim3(p.ntiles, GENERIC_SUBS), dim3(256), stream, (const float*)it.ws, p.nsplit, u.d, scale, out_spec(it));
    return KFAC_OK;
}

static void fbatch_clear(FBatch& b, const kfac_factor_item* dev) {
    b.table = dev;
    b.count = 0;
    b.prefix[0] = 0;
}
static void fbatch_add(FBatch& b, const kfac_factor_item* host, int i, int share, int wgs) {
    b.index[b.count] = i;
    b.share[b.count] = share;
    b.prefix[b.count + 1] = b.prefix[b.count] + wgs;
    if (!b.table) b.single = host[i];
    ++b.count;
}

// All builds of items[0..count): matrix-core builds grouped by kernel variant into batched launches, the rest in one launch and one second
// pass (a lone one by the kernels that look nothing up).  `dev` may be nullptr only when count == 1.
static int run_factor_items(const kfac_factor_item* host, const kfac_factor_item* dev, int count, hipStream_t stream) {
    for (int i = 0; i < count; ++i) {
        Unfold u;
        const int rc = check_item(host[i], &u);
        if (rc != KFAC_OK) return rc;
    }
    const CallCut cut = cut_call(host, count);
    const bool many = cut.many;
    FBatch b, fin[FINISH_LISTS];                       // fin: second passes, after all tiles
    auto finish = [&](int k) -> int {
        const int rc = launch_factor_finish(fin[k], k, stream);
        fbatch_clear(fin[k], dev);
        return rc;
    };
    for (int k = 0; k < FINISH_LISTS; ++k) fbatch_clear(fin[k], dev);
    auto repack = [&]() -> int {
        if (b.count) KFAC_LAUNCH(factor_repack_kernel, dim3(b.prefix[b.count]), dim3(256), stream, b);
        fbatch_clear(b, dev);
        return KFAC_OK;
    };
    fbatch_clear(b, dev);
    for (int i = 0; i < count; ++i) {
        Unfold u;
        View v;
        item_unfold(host[i], &u);
        if (route_of(u, host[i].x, many, &v) != ROUTE_TILE || !v.repack) continue;
        fbatch_add(b, host, i, 0, repack_wgs(u, v));
        if (b.count == FMAXB) {
            int rc = repack();
            if (rc != KFAC_OK) return rc;
        }
    }
    int rc = repack();
    if (rc != KFAC_OK) return rc;
    // kernel variants: tile widths x dtype
    static const struct { bool wide; int dtype; } VAR[5] = {{false, KFAC_BF16}, {false, KFAC_F16}, {true, KFAC_BF16}, {true, KFAC_F16}, {false, KFAC_F32}};
    for (int var = 0; var < 5; ++var) {
        int next = 0;
        while (next < count) {
            fbatch_clear(b, dev);
            struct Pick { int item, share, rows, work, wgs, finish, list; } pick[FMAXB];
            int n = 0, widest = 0;
            bool planes = false;
            for (; next < count && n < FMAXB; ++next) {
                Unfold u;
                View v;
                item_unfold(host[next], &u);
                if (u.dtype != VAR[var].dtype || route_of(u, host[next].x, many, &v) != ROUTE_TILE) continue;
                const int share = cut.share(v);
                if (v.shared) {
                    const SharedPlan p = plan_shared(v, share);
                    if ((p.tw == 256) != VAR[var].wide) continue;
                    widest = std::max(widest, p.tw);
                    pick[n++] = {next, share, p.rows, p.first[4], shared_workgroups(p), shared_assemble_wgs(v),
                                 v.chunked ? FINISH_CHANNELS : FINISH_FEW};
                    continue;
                }
                const FactorPlan p = plan_tiles(v, share);
                if ((p.tw == 256) != VAR[var].wide) continue;
                widest = std::max(widest, p.tw);
                planes = planes || v.planes;
                pick[n++] = {next, share, p.rows_per_split, p.ntiles * p.nsplit, (int)align_up(p.ntiles * p.nsplit, 8),   // (see unit_of)
                             p.nsplit > 1 ? reduce_wgs(v, p) : 0, p.nsplit >= MANY_SPLITS ? FINISH_MANY : FINISH_FEW};
            }
            if (n == 0) continue;
            // the longest workgroups first: the short ones fill the end of the launch
            std::stable_sort(pick, pick + n, [](const Pick& a, const Pick& c) { return a.rows > c.rows; });
            int turn = 0;
            for (int i = 0; i < n; ++i) {
                fbatch_add(b, host, pick[i].item, pick[i].share | turn << SHARE_TURN_SHIFT, pick[i].wgs);
                turn = next_turn(turn, pick[i].work);
            }
            rc = VAR[var].dtype == KFAC_BF16 ? launch_tiles<0>(widest, planes, b, stream)
               : VAR[var].dtype == KFAC_F16 ? launch_tiles<1>(widest, planes, b, stream)
                                            : launch_tiles<2>(widest, planes, b, stream);
            if (rc != KFAC_OK) return rc;
            for (int i = 0; i < n; ++i) {
                if (!pick[i].finish) continue;
                FBatch& f = fin[pick[i].list];
                fbatch_add(f, host, pick[i].item, pick[i].share, pick[i].finish);
                if (f.count == FMAXB && (rc = finish(pick[i].list)) != KFAC_OK) return rc;
            }
        }
    }
    for (int k = 0; k < FINISH_LISTS; ++k)
        if ((rc = finish(k)) != KFAC_OK) return rc;
    FBatch red;                                        // second passes of the generic builds
    auto generic = [&]() -> int {
        if (b.count == 1) {                            // (the kernels that need not look the build up)
            Unfold u;
            item_unfold(host[b.index[0]], &u);
            const int rc = run_generic(u, host[b.index[0]], stream);
            if (rc != KFAC_OK) return rc;
        } else if (b.count) {
            KFAC_LAUNCH(factor_generic_batch_kernel, dim3(b.prefix[b.count]), dim3(256), stream, b);
            if (red.count) KFAC_LAUNCH(factor_reduce_batch_kernel, dim3(red.prefix[red.count]), dim3(256), stream, red);
        }
        fbatch_clear(b, dev);
        fbatch_clear(red, dev);
        return KFAC_OK;
    };
    fbatch_clear(b, dev);
    fbatch_clear(red, dev);
    for (int i = 0; i < count; ++i) {
        Unfold u;
        View v;
        item_unfold(host[i], &u);
        if (route_of(u, host[i].x, many, &v) == ROUTE_TILE) continue;
        const FactorPlan p = plan_generic(u);
        fbatch_add(b, host, i, 0, p.ntiles * p.nsplit);
        if (p.nsplit > 1) fbatch_add(red, host, i, 0, p.ntiles * GENERIC_SUBS);
        if (b.count == FMAXB && (rc = generic()) != KFAC_OK) return rc;
    }
    return generic();
}

}  // namespace kfac

using namespace kfac;

extern "C" size_t kfac_factor_workspace_bytes(int op, const kfac_layer_desc* desc) {
    Unfold u;
    bool ok = op == KFAC_OP_FACTOR_A ? make_unfold_A(desc, &u) : op == KFAC_OP_FACTOR_G ? make_unfold_G(desc, &u) : false;
    if (!ok) return 0;
    return item_ws_bytes(u);
}

static int factor_single(int op, const kfac_layer_desc* desc, const void* x, float scale, float* out, void* ws,
                         size_t ws_bytes, void* stream) {
    if (!desc) return KFAC_ERR_INVALID_ARG;
    kfac_factor_item it;
    it.desc = *desc; it.x = x; it.out = out; it.ws = ws; it.ws_bytes = ws_bytes; it.scale = scale; it.op = op;
    it.running = nullptr; it.decay = 0.f; it.packed = 0;
    return run_factor_items(&it, nullptr, 1, (hipStream_t)stream);
}

extern "C" int kfac_factor_A(const kfac_layer_desc* desc, const void* act, float scale, float* A, void* ws,
                             size_t ws_bytes, void* stream) {
    return factor_single(KFAC_OP_FACTOR_A, desc, act, scale, A, ws, ws_bytes, stream);
}

extern "C" int kfac_factor_G(const kfac_layer_desc* desc, const void* gout, float scale, float* G, void* ws,
                             size_t ws_bytes, void* stream) {
    return factor_single(KFAC_OP_FACTOR_G, desc, gout, scale, G, ws, ws_bytes, stream);
}

extern "C" int kfac_factor_batched(const kfac_factor_item* items_host, const kfac_factor_item* items_dev, int32_t count,
                                   void* stream) {
    if (count == 0) return KFAC_OK;                       // nothing to do, no launch
    if (!items_host || !items_dev || count < 0) return KFAC_ERR_INVALID_ARG;
    return run_factor_items(items_host, items_dev, count, (hipStream_t)stream);
}
