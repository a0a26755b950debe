// Batch Normalization layers (Sec. 5.4): their Fisher matrix is not Kronecker-factorised.  With theta = (scale_1..C,
// shift_1..C), the gradient of sample n is
//     g_n[c] = sum_s gout[n,s,c] * xhat[n,s,c],     g_n[C + c] = sum_s gout[n,s,c]        (s = spatial position)
// and F = (1/N) sum_n g_n g_n^T (2C x 2C), or its diagonal.  This file builds the per-sample gradients from NHWC
// tensors, for all BN layers of a network in one launch per dtype plus one for the sums over chunks (HBM bound:
// both tensors are read once), and applies the diagonal form; the full form is the generic factor build + damped
// inverse + product on the (N x 2C) gradient matrix.
#include <algorithm>

#include "common.h"

namespace kfac {

constexpr int BN_MAX = 64;            // layers per launch (argument block under 4 KB)
// Elements of each tensor per workgroup of the vector kernel, at most, and in one sum: a workgroup's positions are summed in two halves, so that
// chains of additions are as long as with workgroups of half the size (as one sum, errors were up to 1.16 times as large).  The 53 layers of
// ResNet-50 at batch 1, 4 and 32 in bf16 and 8 in fp32, us: workgroups of 32,768 elements 18.8, 37.7, 249 and 119, of 65,536 16.8, 35.6, 235 and
// 118, of 131,072 (as one sum) 18.5, 32.5, 231 and 118, but then single layers take up to 25 % more.
constexpr int BN_UNIT = 65536, BN_SUM = 32768;
constexpr int BN_CVW = 64;            // 16-byte vectors side by side in a workgroup, at most
constexpr int BN_SP_GENERIC = 512;    // positions per workgroup of the general kernel
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// channels of a 16-byte vector
static inline __host__ __device__ int bn_vec(int dtype) { return dtype == KFAC_F32 ? 4 : 8; }

// How one layer is cut into workgroups.  Layers whose channels are whole 16-byte vectors: a workgroup owns `cvw` vectors of
// `sp` consecutive positions of one sample; its 256 threads are cvw vectors x (256 / cvw) position lanes.  General layers: all
// channels of `sp` positions.
struct BnPlan {
    int cvw, ncb, sp, nchunk;
    int half;         // positions in a workgroup's first sum, of two (sp: there is one)
    bool halves;      // a call of few workgroups may give each half to one of its own: the sums, and so the result, are the same
};

// Calls of few workgroups are bound by what one CU reads.  Of inputs that no cache holds, halves apart and whole, us: 64 channels of 56 x 56,
// two samples, fp32 10.8 and 13.7; of 112 x 112 in fp32 13.2 and 17.2, eight samples 20.1 and 26.8, bf16 12.1 and 14.7, 16.1 and 19.4; of 224 x 224
// (49 chunks) fp32 25.1 and 31.1.  With 208 workgroups (112 x 112, 16 samples) halves take 31.2 and 29.2.
constexpr int BN_HALVES_WGS = 128;
static BnPlan bn_plan(int C, int HW, int dtype, bool vec) {
    BnPlan p;
    if (!vec) {
        p.cvw = 0; p.ncb = 1;
        p.nchunk = (HW + BN_SP_GENERIC - 1) / BN_SP_GENERIC;
        p.sp = p.half = BN_SP_GENERIC;
        p.halves = false;
        return p;
    }
    const int cv = C / bn_vec(dtype);
    p.cvw = cv < BN_CVW ? cv : BN_CVW;
    p.ncb = (cv + p.cvw - 1) / p.cvw;
    const int lanes = 256 / p.cvw;
    // (in elements, not bytes)
    int sp = BN_UNIT / (p.cvw * bn_vec(dtype));
    if (sp < 4 * lanes) sp = 4 * lanes;
    p.nchunk = (HW + sp - 1) / sp;
    p.sp = (HW + p.nchunk - 1) / p.nchunk;            // even chunks, no short tail
    // (whole rounds of loads: a second sum then costs none)
    p.half = p.sp * p.cvw * bn_vec(dtype) > BN_SUM ? std::max((p.sp / 2 + 2 * lanes) / (4 * lanes), 1) * (4 * lanes) : p.sp;
    p.half = std::min(p.half, p.sp);
    p.halves = p.half < p.sp && p.nchunk > 1;
    return p;
}

struct BnBatch {
    int count;
    unsigned prefix[BN_MAX + 1];      // first workgroup of layer i
    int C[BN_MAX], HW[BN_MAX], sp[BN_MAX], nchunk[BN_MAX];
    int half[BN_MAX];                 // BnPlan::half; negative: a workgroup has one half of a chunk (nchunk: halves)
    const void* x[BN_MAX];
    const void* gout[BN_MAX];
    float* dst[BN_MAX];               // nchunk == 1: g itself; else the layer's partial sums [n][chunk][2C]
};

struct BnReduceBatch {
    int count;
    unsigned prefix[BN_MAX + 1];      // first workgroup of layer i; one workgroup = 256 columns of one sample
    int C2[BN_MAX];
    int nchunk[BN_MAX];               // negative: that many halves
    const float* partial[BN_MAX];
    float* g[BN_MAX];
};

// NHWC, channels whole vectors.  Both tensors are read once, 16 bytes per thread and load, eight loads in flight.
// (fp32 went through the general kernel before, one 4-byte load after the other: the gradients and the diagonal form of 53 layers
// at batch 2 19.2 ms, now 0.25 ms, most of it the 53 launches.)
// TWO: some layer of the launch has two sums to a workgroup, or halves.  (Asked for each workgroup, this costs launches without any 0.1 to
// 0.2 us: 2,048 channels of 7 x 7 4.2 us instead of 4.0 in fp32, 5.4 instead of 5.2 in bf16.)
template <int DTYPE, bool STREAM, bool TWO>
__global__ __launch_bounds__(256) void bn_partial_kernel(BnBatch b) {
    constexpr int V = DTYPE == KFAC_F32 ? 4 : 8;
    __shared__ float red[(TWO ? 2 : 1) * 256 * 2 * V];   // [sum][position lane][scale, shift][vector][V]
    const int t = threadIdx.x;
    const int m = __syncthreads_count(t < b.count - 1 && b.prefix[t + 1] <= blockIdx.x);
    const int C = b.C[m], HW = b.HW[m], sp = b.sp[m], half = TWO ? abs(b.half[m]) : sp, nchunk = b.nchunk[m];
    const bool halves = TWO && b.half[m] < 0;
    const int cv = C / V;
    const int cvw = cv < BN_CVW ? cv : BN_CVW;
    const int ncb = (cv + cvw - 1) / cvw;
    const int lanes = 256 / cvw;
    unsigned local = blockIdx.x - b.prefix[m];
    const int cb = local % ncb; local /= ncb;
    const int chunk = local % nchunk;
    const int n = local / nchunk;
    const KFAC_AS1 v4u* __restrict__ X = (const KFAC_AS1 v4u*)b.x[m];
    const KFAC_AS1 v4u* __restrict__ G = (const KFAC_AS1 v4u*)b.gout[m];
    const int vec0 = t % cvw, pl = t / cvw;
    const int vec = cb * cvw + vec0;
    const int w8 = cvw * V;                              // channels of this workgroup
    const int first = halves ? chunk >> 1 : chunk, part = halves ? chunk & 1 : 0;
    const int sums = !TWO || halves || half == sp ? 1 : 2;
    int i = 0;
    do {
        const int s0 = min(HW, first * sp + (TWO ? (part + i) * half : 0)), s1 = min(HW, first * sp + (part + i == 0 ? half : sp));
        float ds[V] = {}, db[V] = {};
        if (pl < lanes && vec < cv) {
            const size_t row0 = (size_t)n * HW;
            for (int s = s0 + pl; s < s1; s += 4 * lanes) {
                v4u xv[4], gv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {                // masked, branch free: a position past the end re-reads s
                    const int su = s + u * lanes;
                    const bool ok = su < s1;
                    const size_t at = (row0 + (ok ? su : s)) * cv + vec;
                    xv[u] = STREAM ? __builtin_nontemporal_load(X + at) : X[at];
                    gv[u] = STREAM ? __builtin_nontemporal_load(G + at) : G[at];
                    if (!ok) gv[u] = v4u{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const unsigned xw = xv[u][k], gw = gv[u][k];
                        if constexpr (DTYPE == KFAC_F32) {
                            const float g = __uint_as_float(gw);
                            ds[k] = fmaf(g, __uint_as_float(xw), ds[k]);
                            db[k] += g;
                            continue;
                        }
                        float x0, x1, g0, g1;
                        if constexpr (DTYPE == KFAC_F16) {
                            x0 = half_bits_to_float((uint16_t)(xw & 0xffff)); x1 = half_bits_to_float((uint16_t)(xw >> 16));
                            g0 = half_bits_to_float((uint16_t)(gw & 0xffff)); g1 = half_bits_to_float((uint16_t)(gw >> 16));
                        } else {
                            x0 = __uint_as_float(xw << 16); x1 = __uint_as_float(xw & 0xffff0000u);
                            g0 = __uint_as_float(gw << 16); g1 = __uint_as_float(gw & 0xffff0000u);
                        }
                        ds[2 * k % V] = fmaf(g0, x0, ds[2 * k % V]);             db[2 * k % V] += g0;
                        ds[(2 * k + 1) % V] = fmaf(g1, x1, ds[(2 * k + 1) % V]); db[(2 * k + 1) % V] += g1;
                    }
            }
        }
        if (pl < lanes) {
            float* to = red + i * (lanes * 2 * w8) + pl * 2 * w8 + vec0 * V;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                to[e] = ds[e];
                to[w8 + e] = db[e];
            }
        }
    } while (++i < sums);
    // sum over the position lanes in a fixed order; every thread takes part
    __syncthreads();
    gfloat* dst = as_global(b.dst[m]) + ((size_t)n * nchunk + chunk) * (2 * C);
    for (int e = t; e < 2 * w8; e += 256) {
        float a = red[e];
        if (sums == 2) {                                 // (side by side: each is a chain of LDS reads)
            const float* second = red + lanes * 2 * w8;
            float a2 = second[e];
            for (int q = 1; q < lanes; ++q) {
                a += red[q * 2 * w8 + e];
                a2 += second[q * 2 * w8 + e];
            }
            a += a2;
        } else {
            for (int q = 1; q < lanes; ++q) a += red[q * 2 * w8 + e];
        }
        const int half = e >= w8, c = cb * w8 + (e - half * w8);
        if (c < C) dst[half * C + c] = a;
    }
}

// any dtype / channel count: thread = one channel, slow but general
__global__ __launch_bounds__(256) void bn_partial_generic_kernel(const void* xhat_, const void* gout_, int dtype, int C,
                                                                 int HW, int nchunk, float* partial_) {
    gfloat* __restrict__ partial = as_global(partial_);
    const int n = blockIdx.y, chunk = blockIdx.x;
    const int s0 = chunk * BN_SP_GENERIC, s1 = min(HW, s0 + BN_SP_GENERIC);
    auto at = [&](const void* p, size_t i) -> float {
        if (dtype == KFAC_F32) return ((const KFAC_AS1 float*)p)[i];
        const uint16_t b = ((const KFAC_AS1 uint16_t*)p)[i];
        return dtype == KFAC_BF16 ? bf16_bits_to_float(b) : half_bits_to_float(b);
    };
    for (int c = threadIdx.x; c < C; c += 256) {
        float ds = 0.f, db = 0.f;
        for (int s = s0; s < s1; ++s) {
            const size_t i = ((size_t)n * HW + s) * C + c;
            const float g = at(gout_, i);
            ds = fmaf(g, at(xhat_, i), ds);
            db += g;
        }
        gfloat* dst = partial + ((size_t)n * nchunk + chunk) * (2 * C);
        dst[c] = ds;
        dst[C + c] = db;
    }
}

// g[n][j] = sum over chunks, fixed order
__global__ __launch_bounds__(256) void bn_reduce_kernel(BnReduceBatch b) {
    const int t = threadIdx.x;
    const int m = __syncthreads_count(t < b.count - 1 && b.prefix[t + 1] <= blockIdx.x);
    const int C2 = b.C2[m], nchunk = abs(b.nchunk[m]);
    const int cblocks = (C2 + 255) >> 8;
    const unsigned local = blockIdx.x - b.prefix[m];
    const int n = local / cblocks, j = (local % cblocks) * 256 + t;
    if (j >= C2) return;
    const gfloat* __restrict__ partial = as_global(b.partial[m]);
    float s = 0.f;
    auto at = [&](int q) { return partial[((size_t)n * nchunk + q) * C2 + j]; };
    if (b.nchunk[m] < 0)                                     // (an even number)
        for (int q = 0; q < nchunk; q += 2) s += at(q) + at(q + 1);
    else
        for (int q = 0; q < nchunk; ++q) s += at(q);
    as_global(b.g[m])[(size_t)n * C2 + j] = s;
}

// diag(F)[j] = (1/N) sum_n g[n][j]^2 ;  out[j] = grad[j] / (diag(F)[j] + damping)
// A small, latency-bound launch (one per layer): 64 columns x 4 groups of samples per workgroup, eight loads in flight per
// thread, so that 32 samples cost one trip to memory (9.4 us with one thread walking down a column).
__global__ __launch_bounds__(256) void bn_diag_kernel(const float* g_, int N, int C2, const float* grad, float damping,
                                                      float* fisher_diag, float* out) {
    __shared__ float part[3][64];
    const gfloat* __restrict__ g = as_global(g_);
    const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + lane, jc = min(j, C2 - 1);
    const float gr = grp == 0 && out ? as_global(grad)[jc] : 0.f;
    float s = 0.f;
    for (int n0 = grp; n0 < N; n0 += 32) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = g[(size_t)min(n0 + 4 * k, N - 1) * C2 + jc];
#pragma unroll
        for (int k = 0; k < 8; ++k) s = n0 + 4 * k < N ? fmaf(v[k], v[k], s) : s;
    }
    if (grp > 0) part[grp - 1][lane] = s;
    __syncthreads();
    if (grp > 0 || j >= C2) return;
    s = (s + part[0][lane]) + (part[1][lane] + part[2][lane]);
    s /= (float)N;
    if (fisher_diag) fisher_diag[j] = s;
    if (out) out[j] = gr / (s + damping);
}

}  // namespace kfac

using namespace kfac;

static bool bn_item_ok(const kfac_bn_item& it) {
    if (!it.xhat || !it.gout || !it.g) return false;
    if (it.N <= 0 || it.C <= 0 || it.HW <= 0 || it.N > 65535 || it.C > 16384) return false;
    if (it.dtype != KFAC_F32 && it.dtype != KFAC_BF16 && it.dtype != KFAC_F16) return false;
    return (long long)it.N * it.C * it.HW <= 0x7fffffffLL;
}

static bool bn_item_vec(const kfac_bn_item& it) {
    return it.C % bn_vec(it.dtype) == 0 && (((uintptr_t)it.xhat | (uintptr_t)it.gout) & 15) == 0;
}

// bytes of partial sums one layer needs (none when a single chunk covers all positions).  Neither the 16-byte alignment of the
// tensors nor the call's other layers are known when only the shape is, nor, of a single layer, the dtype: every cutting is covered.
static size_t bn_item_ws(int N, int C, int HW, int dtype) {
    int nchunk = bn_plan(C, HW, dtype, false).nchunk;
    for (int dt : {dtype, (int)KFAC_F32, (int)KFAC_BF16})
        if (C % bn_vec(dtype) == 0 && C % bn_vec(dt) == 0) {
            const BnPlan p = bn_plan(C, HW, dt, true);
            nchunk = std::max(nchunk, p.halves ? 2 * p.nchunk : p.nchunk);
        }
    return nchunk > 1 ? align_up((size_t)N * nchunk * 2 * C * sizeof(float), 256) : 0;
}

extern "C" size_t kfac_bn_sample_grads_batched_workspace_bytes(const kfac_bn_item* items_host, int32_t count) {
    if (!items_host || count <= 0) return 0;
    size_t total = 0;
    for (int i = 0; i < count; ++i) {
        const kfac_bn_item& it = items_host[i];
        if (it.N <= 0 || it.C <= 0 || it.HW <= 0) return 0;
        total += bn_item_ws(it.N, it.C, it.HW, it.dtype);
    }
    return total;
}

extern "C" int kfac_bn_sample_grads_batched(const kfac_bn_item* items_host, int32_t count, void* ws, size_t ws_bytes,
                                            void* stream) {
    if (!items_host || count < 0) return KFAC_ERR_INVALID_ARG;
    if (count == 0) return KFAC_OK;
    for (int i = 0; i < count; ++i)
        if (!bn_item_ok(items_host[i])) return KFAC_ERR_INVALID_ARG;
    const size_t need = kfac_bn_sample_grads_batched_workspace_bytes(items_host, count);
    if (need && (!ws || ((uintptr_t)ws & 255) || ws_bytes < need)) return KFAC_ERR_WORKSPACE;
    char* wsp = (char*)ws;
    for (int first = 0; first < count; first += BN_MAX) {
        const int cnt = count - first < BN_MAX ? count - first : BN_MAX;
        BnBatch lists[3];                                 // the fp32, bf16 and fp16 layers of this group
        BnReduceBatch rb;
        unsigned wgs[3] = {0, 0, 0}, nred = 0;
        bool two[3] = {false, false, false};
        size_t bytes[3] = {0, 0, 0};                      // of both tensors
        lists[KFAC_F32].count = lists[KFAC_BF16].count = lists[KFAC_F16].count = rb.count = 0;
        long long whole = 0;                              // workgroups with whole chunks
        for (int i = 0; i < cnt; ++i) {
            const kfac_bn_item& it = items_host[first + i];
            const BnPlan p = bn_plan(it.C, it.HW, it.dtype, bn_item_vec(it));
            whole += (long long)it.N * p.nchunk * p.ncb;
        }
        for (int i = 0; i < cnt; ++i) {
            const kfac_bn_item& it = items_host[first + i];
            const bool vec = bn_item_vec(it);
            BnPlan p = bn_plan(it.C, it.HW, it.dtype, vec);
            const bool halves = p.halves && whole <= BN_HALVES_WGS;
            if (halves) p.nchunk *= 2;
            float* dst = it.g;
            if (p.nchunk > 1) {
                dst = (float*)wsp;
                const int k = rb.count++;
                rb.prefix[k] = nred;
                rb.C2[k] = 2 * it.C; rb.nchunk[k] = halves ? -p.nchunk : p.nchunk; rb.partial[k] = dst; rb.g[k] = it.g;
                nred += (unsigned)it.N * ((2 * it.C + 255) / 256);
            }
            wsp += bn_item_ws(it.N, it.C, it.HW, it.dtype);
            if (vec) {
                BnBatch& b = lists[it.dtype];
                unsigned& units = wgs[it.dtype];
                const int k = b.count++;
                b.prefix[k] = units;
                b.C[k] = it.C; b.HW[k] = it.HW; b.sp[k] = p.sp; b.half[k] = halves ? -p.half : p.half; b.nchunk[k] = p.nchunk;
                b.x[k] = it.xhat; b.gout[k] = it.gout; b.dst[k] = dst;
                units += (unsigned)it.N * p.nchunk * p.ncb;
                two[it.dtype] |= p.half < p.sp;
                bytes[it.dtype] += (size_t)it.N * it.C * it.HW * (it.dtype == KFAC_F32 ? 8 : 4);
            } else {
                KFAC_LAUNCH(bn_partial_generic_kernel, dim3(p.nchunk, it.N), dim3(256), (hipStream_t)stream, it.xhat, it.gout,
                            (int)it.dtype, (int)it.C, (int)it.HW, p.nchunk, dst);
            }
        }
        for (int dt = 0; dt < 3; ++dt) {
            BnBatch& b = lists[dt];
            if (b.count == 0) continue;
            b.prefix[b.count] = wgs[dt];
#define KFAC_BN_LAUNCH_AS(DTYPE, NAME, STREAM, TWO)                                                                                 \
    KFAC_LAUNCH_AS("bn_partial_kernel<" #DTYPE NAME ">", (bn_partial_kernel<DTYPE, STREAM, TWO>), dim3(wgs[dt]), dim3(256), (hipStream_t)stream, b)
#define KFAC_BN_LAUNCH(DTYPE)                                                                                                       \
    do {                                                                                                                            \
        if (bytes[dt] > STREAM_BYTES) {                                                                                             \
            if (two[dt]) KFAC_BN_LAUNCH_AS(DTYPE, ", stream", true, true);                                                \
            else KFAC_BN_LAUNCH_AS(DTYPE, ", stream", true, false);                                                                 \
        } else {                                                                                                                    \
            if (two[dt]) KFAC_BN_LAUNCH_AS(DTYPE, "", false, true);                                                       \
            else KFAC_BN_LAUNCH_AS(DTYPE, "", false, false);                                                                        \
        }                                                                                                                           \
    } while (0)
            if (dt == KFAC_F32) KFAC_BN_LAUNCH(KFAC_F32);
            else if (dt == KFAC_BF16) KFAC_BN_LAUNCH(KFAC_BF16);
            else KFAC_BN_LAUNCH(KFAC_F16);
#undef KFAC_BN_LAUNCH_AS
#undef KFAC_BN_LAUNCH
        }
        if (rb.count) {
            rb.prefix[rb.count] = nred;
            KFAC_LAUNCH(bn_reduce_kernel, dim3(nred), dim3(256), (hipStream_t)stream, rb);
        }
    }
    return KFAC_OK;
}

extern "C" size_t kfac_bn_sample_grads_workspace_bytes(int32_t N, int32_t C, int32_t HW) {
    if (N <= 0 || C <= 0 || HW <= 0) return 0;
    return std::max(bn_item_ws(N, C, HW, KFAC_BF16), bn_item_ws(N, C, HW, KFAC_F32));
}

extern "C" int kfac_bn_sample_grads(const void* xhat, const void* gout, int32_t N, int32_t C, int32_t HW, int32_t dtype,
                                    float* g, void* ws, size_t ws_bytes, void* stream) {
    const kfac_bn_item it = {xhat, gout, g, N, C, HW, dtype};
    return kfac_bn_sample_grads_batched(&it, 1, ws, ws_bytes, stream);
}

extern "C" int kfac_bn_diag_precondition(const float* g, int32_t N, int32_t C2, const float* grad, float damping,
                                         float* fisher_diag, float* out, void* stream) {
    if (!g || N <= 0 || C2 <= 0 || (!fisher_diag && !out) || (out && !grad)) return KFAC_ERR_INVALID_ARG;
    if (!(damping >= 0.f)) return KFAC_ERR_INVALID_ARG;
    KFAC_LAUNCH(bn_diag_kernel, dim3((C2 + 63) / 64), dim3(256), (hipStream_t)stream, g, N, C2, grad, damping, fisher_diag, out);
    return KFAC_OK;
}
