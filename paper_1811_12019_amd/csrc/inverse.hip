// Damped inverse of symmetric positive definite factors: Minv = (S + lambda I)^-1  (Sec. 4.2 damping, Eq. 6;
// Algorithm 1 stage 4), fp32.
//
// Method: blocked symmetric sweep (block Gauss-Jordan without pivoting, which is safe for SPD matrices).
// With the matrix cut into 128-wide blocks, eliminating block k does
//     P        = W_kk^-1                       (one workgroup, register resident)
//     T        = W_:k P                        (panel, MFMA)
//     W_ij    -= T_i W_jk^T   for i, j != k    (rank-128 update of the whole matrix, MFMA)
//     W_:k = T, W_k: = T^T, W_kk = -P
// and after all blocks W = -M^-1; the sign flip is folded into the last step.  Every step touches the whole
// matrix, so all steps expose the same, large amount of parallelism, and a batch of matrices of different sizes
// advances together: one launch per stage per step for the whole batch (the workgroup -> (matrix, tile) map is a
// prefix table passed in the kernel arguments).
//
// Launch structure.  The elimination is a chain, 37 steps long for a 4609-wide factor, most of whose steps leave the chip nearly
// idle, so a step is one launch and the bulk of the flops is moved off the chain.  The launch of step k starts from P_k and from
// panel k (block column k, assembled: U_k), both left by the launch before, and has workgroups of three kinds:
//   * the look-ahead pivot: the rank-128 update of the diagonal tile that is pivot block k + 1, with a T_(k+1) = U_(k+1) P_k of its
//     own, kept in registers, and its inversion: P_(k+1);
//   * slabs, half a slab (64 rows) each: T_I = U_I P_k and, from it, the next panel, U_I(k+1) = W_I(k+1) - ... - T_I U_(k+1)^T
//     (U_(k+1) is part of panel k: nothing in the launch waits for another workgroup of it);
//   * tiles of the rest of the matrix, which receive the updates of finished steps in one visit for a group of GM steps (Plan).
// Every matrix of a batch carries its own stage, so that matrices with fewer blocks spread their launches over those of the
// largest one.  The last step's panel is a launch, and one launch for the whole batch writes the outputs (inv_out_kernel).
// Bound: one matrix alone by the look-ahead pivot's workgroup (loads 2.9 us, its T 4.9, update 5.3, the sweep 10, write-out 1.9, from
// launch to launch 1.7; half slabs are done after 12 to 23): 26 us a step, 31 with a sweep of 15.3, 40 when panel and tiles were launches
// of their own.  One matrix alone, us, with the sweep of 15.3 and now: 145 columns 62 and 58, 1000 270 and 240, 2049 530 and 468, 4609 1236
// and 1159; ten ragged ones (10 to 1153 columns) with their preconditioning 393 and 361.  Batches of wide matrices are bound by their tile visits.
// Products: the panel on the bf16 matrix cores with operands split three ways; the updates on the fp16 matrix cores
// from operands that the panel launch has already scaled per half slab (64 rows) and split two ways, stored as planes that
// go to LDS by DMA (gemm_split.h); both to fp32 accuracy.
//
// Storage.  The sweep works on a copy W of the matrix in the caller's workspace that holds only the tiles on and below the diagonal,
// each as the matrix cores leave it in their registers (WsView::tile): a tile is loaded and stored 16 bytes a lane, a quarter of the
// memory instructions of a row-major copy.  (A CU stores four lanes a cycle, whatever a lane stores.)  Tiles at the matrix's edge
// are padded with zeros, which all products leave zero.  The part of block column k above the pivot block is read, transposed, from
// block row k.  Only the last launch writes the caller's dense output, both triangles, exactly symmetric (the upper one is a copy of
// the lower one).
#include "gemm_split.h"
#include "inverse_plan.h"

namespace kfac {

constexpr int MAXB = 64;         // matrices per launch of the kernels that read S (bounded by the 4 KB of kernel arguments)
constexpr int CMAXB = 112;       // matrices per launch of the sweep's per-step kernels, whose argument block is leaner
constexpr int UPD_WAVES = 3;     // wavefronts per SIMD the update kernel is compiled for (register budget)
constexpr int SLD_T = 129;       // staging stride (floats) where the stage is also read column-wise
constexpr int PH = NB / 2;       // rows of a half slab
constexpr int UPD_LDS_BYTES = 48 * 1024;   // of a workgroup of the sweep's launches: three of them on a CU

// Everything a launch needs to know about its matrices travels in the kernel arguments (scalar loads, no dependent
// memory round trip at the start of every workgroup).
struct Batch {
    int count;                        // matrices in this launch
    int prefix[MAXB + 1];             // workgroup prefix sums over them
    int dim[MAXB];
    float damping[MAXB];
    const float* damping_dev[MAXB];   // NULL, or where the damping is to be read from instead
    const float* S[MAXB];
    float* Minv[MAXB];
    void* ws[MAXB];
    int32_t* info[MAXB];
};

static_assert(sizeof(Batch) <= 4096, "the batch travels in the kernel arguments");

// The same for the panel and update launches of the sweep, which no longer need the input matrix or the damping: more
// matrices per launch, i.e. fewer, fuller launches for a batch of many small matrices.
struct ChainBatch {
    int count;
    int prefix[CMAXB + 1];
    int dim[CMAXB];
    int stage[CMAXB];                 // the stage this launch takes for the matrix (plan_of), or -1: none
    float* Minv[CMAXB];
    void* ws[CMAXB];
    int32_t* info[CMAXB];
};
static_assert(sizeof(ChainBatch) <= 4096, "the batch travels in the kernel arguments");

// One matrix of the batch as the kernels see it: pointers typed as global memory.
struct Item {
    const gfloat* S;
    gfloat* Minv;
    gfloat* ws;
    gint* info;
    int dim;
    float damping;
};

__device__ __forceinline__ Item get_item(const Batch& b, int m) {
    Item it;
    it.S = as_global(b.S[m]);
    it.Minv = as_global(b.Minv[m]);
    it.ws = as_global((float*)b.ws[m]);
    it.info = as_global((int*)b.info[m]);
    it.dim = b.dim[m];
    it.damping = b.damping_dev[m] ? *as_global(b.damping_dev[m]) : b.damping[m];
    return it;
}

__device__ __forceinline__ Item get_item(const ChainBatch& b, int m) {
    Item it;
    it.S = nullptr;
    it.Minv = as_global(b.Minv[m]);
    it.ws = as_global((float*)b.ws[m]);
    it.info = as_global((int*)b.info[m]);
    it.dim = b.dim[m];
    it.damping = 0.f;
    return it;
}

// Which matrix workgroup `wg` of a launch belongs to (prefix[m] <= wg < prefix[m + 1]) and its index inside it.
// Every thread compares one prefix entry and the workgroup counts the matrices that end at or before wg: one vector
// load and one barrier instead of a binary search of dependent scalar loads (2 us at the start of every workgroup).
// Must be called by all threads of the workgroup.
template <class B>
__device__ __forceinline__ void locate(const B& b, int wg, int& m, int& local) {
    const int t = threadIdx.x;
    m = __syncthreads_count(t < b.count - 1 && b.prefix[t + 1] <= wg);
    local = wg - b.prefix[m];
}

static inline __host__ __device__ size_t working_copy_floats(int dim) { return (size_t)nblk_of(dim) * (nblk_of(dim) + 1) / 2 * NB * NB; }

// Optional second form of the result, for the products that consume the inverse (preconditioning): the matrix cut
// into 128 x 128 blocks (zero padded), every element scaled by one power of two and split into two fp16 pieces, as two
// planes of n x n blocks in the layout of gemm_split.h (block (s, c) at (s n + c) PRE_SLAB bytes) followed by n x n
// floats that all hold the scale.  The scale: the damped matrix is S + lambda I with S positive semidefinite, so no
// entry of the inverse exceeds 1 / lambda in magnitude; 2^(8 + floor(log2 lambda)) maps that bound to at most 2^8, which
// leaves fp16's range seven more binades before overflow and keeps all 22 bits of entries down to 2^-11 of the bound
// (smaller ones lose bits only below 2^-33 of it).
static inline __host__ __device__ size_t inverse_plane_bytes(int dim) { return (size_t)nblk_of(dim) * nblk_of(dim) * PRE_SLAB; }
static inline __host__ __device__ size_t inverse_planes_bytes(int dim) {
    return 2 * inverse_plane_bytes(dim) + sizeof(float) * nblk_of(dim) * nblk_of(dim);
}
__device__ __forceinline__ float inverse_plane_scale(float damping) {
    return damping > 0.f ? ldexpf(1.0f, 8 + ilogbf(damping)) : 1.0f;
}
// Panels of one step, kept in buffer (step % NBUF): the fp32 copy U of block column k as it was before the step (all
// rows, assembled from both triangles), the fp32 product T = U P, and the scaled fp16 pieces of both (the negated T and
// U, each as a plane of high and a plane of low pieces in the layout of gemm_split.h), which the tile updates multiply.
struct WsView {
    gfloat* W;      // working copy: lower tiles row by row, 64 KB each: 4 x 4 blocks of 32 x 32, float 256 q + 4 lane + i of a block
                    // being row 8 q + 4 (lane / 32) + i, column lane % 32
    gfloat* buf0;   // NBUF panel buffers, `stride` floats each: U | T | -T high | -T low | U high | U low
    size_t stride;
    size_t plane;   // bytes of one piece plane (d_pad x NB fp16)
    gfloat* P0;     // 2 x NB x NB : inverses of the pivot blocks of even and of odd steps
    gfloat* SC;     // 2 NBUF x 2 nblk: power-of-two scales of the half slabs (64 rows) of T and U of every buffer (gemm_split.h)
    int nblk;
    __device__ __forceinline__ gfloat* tile(int I, int J) const { return W + (size_t)(I * (I + 1) / 2 + J) * (NB * NB); }
    __device__ __forceinline__ gfloat* P(int step) const { return P0 + (step & 1) * (NB * NB); }
    __device__ __forceinline__ gfloat* U(int q) const { return buf0 + q * stride; }
    __device__ __forceinline__ gfloat* T(int q) const { return buf0 + q * stride + plane / 2; }
    __device__ __forceinline__ KFAC_AS1 unsigned char* TH(int q) const { return (KFAC_AS1 unsigned char*)(buf0 + q * stride + plane); }
    __device__ __forceinline__ KFAC_AS1 unsigned char* UH(int q) const { return TH(q) + 2 * plane; }
    __device__ __forceinline__ gfloat& scaleT(int q, int half_slab) const { return SC[(q * 2 + 0) * 2 * nblk + half_slab]; }
    __device__ __forceinline__ gfloat& scaleU(int q, int half_slab) const { return SC[(q * 2 + 1) * 2 * nblk + half_slab]; }
};

static inline __host__ __device__ size_t panel_buffer_floats(int dim) { return (size_t)nblk_of(dim) * NB * NB * 4; }

__device__ inline WsView ws_view(gfloat* ws, int dim) {
    const size_t d_pad = (size_t)nblk_of(dim) * NB;
    WsView v;
    v.nblk = nblk_of(dim);
    v.W = ws;
    v.buf0 = v.W + working_copy_floats(dim);
    v.stride = panel_buffer_floats(dim);                 // 2 fp32 panels + 4 fp16 planes = 4 d_pad NB floats
    v.plane = d_pad * NB * 2;
    v.P0 = v.buf0 + NBUF * v.stride;
    v.SC = v.P0 + (size_t)2 * NB * NB;
    return v;
}

// 32 x 32 block (rb, cb) of a tile of W, and a block from / to the accumulators.
__device__ __forceinline__ gfloat* tile_block(gfloat* tile, int rb, int cb) { return tile + (rb * 4 + cb) * 1024; }
__device__ __forceinline__ void load_block(const gfloat* blk, v16f& acc) {
    const gfloat* src = blk + (threadIdx.x & 63) * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const v4f x = *(const KFAC_AS1 v4f*)(src + q * 256);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[4 * q + i] = x[i];
    }
}
__device__ __forceinline__ void store_block(gfloat* blk, const v16f& acc) {
    gfloat* dst = blk + (threadIdx.x & 63) * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) *(KFAC_AS1 v4f*)(dst + q * 256) = v4f{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
}

// ---- pivot block -----------------------------------------------------------------------------------------------
// Inverse of the (at most 128 x 128) pivot block by a symmetric sweep in 16-wide sub-blocks.  The lower triangle of the
// block D lives in registers as 16 x 16 blocks in MFMA accumulator layout (lane l holds rows 4 (l / 16) + i of column l % 16), three
// wavefronts owning whole block rows (PIV_ROW), which deals the products out evenly; wavefront 1 looks ahead: it inverts the next
// 16 x 16 diagonal sub-block while the others update D.  Per sub-block j, one barrier:
//   * wavefronts 0, 2, 3: T16 = U16 . P16 for their own rows (U16 = D's columns j, in LDS) and, straight from these registers,
//     D -= T16 . U16^T on the matrix cores; columns / rows j of D become T16, the sub-block itself -P16 (row j, which needs other
//     wavefronts' T16, a round later); columns / rows j + 1 and diagonal sub-block j + 2 go to LDS for the next round;
//   * wavefront 1: takes sub-block j + 1, which the round before left in LDS, through this round's update, with a T16 of its own,
//     and inverts it.
// Padding with the identity makes ragged blocks (fewer than 128 rows) need no special cases.
// One workgroup, bound by its chain of dependent steps: 3,100 cycles a sub-block, the time of wavefront 1, of which the inversion is
// 2,450 (less 200 since its columns are spread in pairs); the owners are done after 1,300 to 3,000.  4,100 with 32 x 32 blocks in quadrants (one wavefront had 16 of 40 to update), two
// barriers and a rank-1 update per elimination; a loop over the sub-blocks that is not unrolled takes 4,100 too (branches, copies).
constexpr int PSB = 16;          // sub-block
constexpr int PLD = 20;          // LDS row stride of the 16-wide panels (float4 aligned)

// x of lane S of the lane's own row of 16 lanes
template <int S>
__device__ __forceinline__ float row_bcast(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + S, 0xf, 0xf, true));
}
// x and y of the same lane of row G (of the four rows of 16 lanes), in every row
template <int G>
__device__ __forceinline__ void group_bcast2(float& x, float& y) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);   // x's rows 0 1, y's 0 1 / 2 3, 2 3
    const unsigned r = a[G >> 1];
    const auto b = __builtin_amdgcn_permlane16_swap(r, r, false, false);                                     // the even / the odd one, twice each
    const unsigned q = b[G & 1];
    const auto c = __builtin_amdgcn_permlane32_swap(q, q, false, false);
    x = __uint_as_float(c[0]);
    y = __uint_as_float(c[1]);
}

__device__ __forceinline__ float rsqrt_newton(float p) {
    const float r = __builtin_amdgcn_rsqf(p);              // 1 ulp estimate + one Newton step
    return fmaf(0.5f * r, fmaf(-p * r, r, 1.0f), r);
}

// Four elimination steps of invert16_wave, columns 4 S .. + 3; N: minus the matrix E that is swept.  With L the Cholesky factor of the 4 x 4
// pivot block (formed by all lanes alike) and W = V L^-T, V being the four columns of E with minus the identity in the pivot rows, all that
// the sweep does is E - W W^T, where E counts as zero in the pivot rows and columns: -V P V^T beside them, V P and P V^T in them, -P where
// they cross.  One matrix-core product, and the same bits on both sides of the diagonal: E stays symmetric.  (Rows and columns that drift
// apart by rounding cost an ill-conditioned block most of its accuracy.)  It is added to N, which the matrix core does one elimination after
// the other: what each leaves is rounded at its own size.  Their sum, formed first, is rounded at the size of what cancels: inverses of up to 16
// columns with condition numbers from 1e4 on erred 1.1 to 1.7 times as much.
template <int S>
__device__ __forceinline__ void invert16_step4(v4f& N, int i, int g, const float (&unit)[4], float (&piv)[16]) {
    float v[4], u[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = N[q];
    group_bcast2<S>(v[0], v[1]);                                      // N(i, 4 S + q)
    group_bcast2<S>(v[2], v[3]);
    const float a00 = -row_bcast<4 * S>(v[0]);
    float a10 = -row_bcast<4 * S + 1>(v[0]), a20 = -row_bcast<4 * S + 2>(v[0]), a30 = -row_bcast<4 * S + 3>(v[0]);
    float a11 = -row_bcast<4 * S + 1>(v[1]), a21 = -row_bcast<4 * S + 2>(v[1]), a31 = -row_bcast<4 * S + 3>(v[1]);
    float a22 = -row_bcast<4 * S + 2>(v[2]), a32 = -row_bcast<4 * S + 3>(v[2]), a33 = -row_bcast<4 * S + 3>(v[3]);
    const bool prow = (i >> 2) == S;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = prow ? unit[q] : v[q];         // -V
    const float r0 = rsqrt_newton(a00);
    a10 *= r0; a20 *= r0; a30 *= r0;
    a11 = fmaf(-a10, a10, a11); a21 = fmaf(-a20, a10, a21); a31 = fmaf(-a30, a10, a31);
    a22 = fmaf(-a20, a20, a22); a32 = fmaf(-a30, a20, a32); a33 = fmaf(-a30, a30, a33);
    u[0] = -v[0] * r0;
    const float r1 = rsqrt_newton(a11);
    a21 *= r1; a31 *= r1;
    a22 = fmaf(-a21, a21, a22); a32 = fmaf(-a31, a21, a32); a33 = fmaf(-a31, a31, a33);
    u[1] = fmaf(-a10, u[0], -v[1]) * r1;
    const float r2 = rsqrt_newton(a22);
    a32 *= r2;
    a33 = fmaf(-a32, a32, a33);
    u[2] = fmaf(-a21, u[1], fmaf(-a20, u[0], -v[2])) * r2;
    const float r3 = rsqrt_newton(a33);
    u[3] = fmaf(-a32, u[2], fmaf(-a31, u[1], fmaf(-a30, u[0], -v[3]))) * r3;
    piv[4 * S] = a00; piv[4 * S + 1] = a11; piv[4 * S + 2] = a22; piv[4 * S + 3] = a33;
    const float lo = (g & 1) ? u[1] : u[0], hi = (g & 1) ? u[3] : u[2], w = (g & 2) ? hi : lo;
    const bool gone = prow || g == S;
    v4f rest;
#pragma unroll
    for (int q = 0; q < 4; ++q) rest[q] = gone ? 0.f : N[q];
    N = __builtin_amdgcn_mfma_f32_16x16x4f32(w, w, rest, 0, 0, 0);
}

// One wavefront: Ps = inverse of the symmetric positive definite 16 x 16 block whose element (i, 4 g + q), negated, lane
// (i = lane % 16, g = lane / 16) holds in N[q] (of two that mirror each other the lower one counts); N becomes the inverse.
// Returns the 1-based index of the first non-positive pivot, or 0.  Nothing goes through LDS on the way.
__device__ __forceinline__ int invert16_wave(v4f& N, float* Ps) {
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    float piv[16], unit[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) unit[q] = (i & 3) == q ? 1.f : 0.f;
    invert16_step4<0>(N, i, g, unit, piv);
    invert16_step4<1>(N, i, g, unit, piv);
    invert16_step4<2>(N, i, g, unit, piv);
    invert16_step4<3>(N, i, g, unit, piv);
    *(v4f*)&Ps[i * PLD + 4 * g] = N;
    if (piv[15] > 0.f) return 0;                           // (a pivot that is not positive makes all later ones NaN)
    int bad = 0;
#pragma unroll
    for (int s = 15; s >= 0; --s) bad = piv[s] > 0.f ? bad : s + 1;
    return bad;
}

// LDS of the pivot code: the sweep's panels (U16, T16, P16 and a diagonal sub-block, of two rounds each); before and after
// it, in the same memory, the block's packed lower triangle (row r holds columns 0..r).
constexpr int TRI_FLOATS = NB * (NB + 1) / 2;
constexpr int PIV_US = 0, PIV_TS = 2 * NB * PLD, PIV_PS = 4 * NB * PLD, PIV_DG = PIV_PS + 2 * PSB * PLD,
              PIV_BAD = PIV_DG + 2 * PSB * PSB;
constexpr int PIV_LDS_FLOATS = PIV_BAD + 4;
static_assert(TRI_FLOATS <= PIV_LDS_FLOATS, "one buffer serves both uses");

__device__ __forceinline__ int tri_at(int r, int c) { return ((r * (r + 1)) >> 1) + c; }          // r >= c
__device__ __forceinline__ int tri_sym(int r, int c) { return r >= c ? tri_at(r, c) : tri_at(c, r); }

// Block rows of the three owners (wavefronts 0, 2, 3): 7 4 / 6 3 0 / 5 2 1, which are 13, 12 and 11 blocks to update and 2, 3 and 3 of
// T16 to form: 15, 15 and 14 products of 16 x 16 x 16.  (Quadrants of 32 x 32 blocks left one wavefront with 16 of 40.)
constexpr int PIV_BLOCKS = 13;
constexpr int piv_rows(int role) { return role == 0 ? 2 : 3; }
constexpr int piv_row(int role, int x) { return x == 0 ? 7 - role : x == 1 ? 4 - role : role - 1; }
constexpr int piv_slot(int role, int x) { return x == 0 ? 0 : piv_slot(role, x - 1) + piv_row(role, x - 1) + 1; }
static_assert(piv_slot(0, 2) == 13 && piv_slot(1, 3) == 12 && piv_slot(2, 3) == 11, "all 36 blocks, no more than a wavefront holds");
typedef v4f PivotBlocks[PIV_BLOCKS];

#define KFAC_INLINE __attribute__((always_inline))
template <int V> struct Int { static constexpr int value = V; constexpr operator int() const { return V; } };
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {                      // f(Int<0>()), ..: registers want constant indices
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(Int<N - 1>());
    }
}
template <class F>
__device__ __forceinline__ void with_role(int wave, F&& f) {             // wave: uniform; nothing for wavefront 1
    if (wave == 0) f(Int<0>());
    else if (wave == 2) f(Int<1>());
    else if (wave == 3) f(Int<2>());
}
// f(block row, block column, the block) for every block of the wavefront (row and column: uniform values, so that all owners share the
// code and a register has the same index in it)
template <class F>
__device__ __forceinline__ void each_block(int wave, PivotBlocks& D, F&& f) {
    if (wave == 1) return;
    const int role = max(0, wave - 1), r0 = 7 - role, r1 = 4 - role, r2 = role - 1;      // (piv_row)
    static_for<PIV_BLOCKS>([&](auto slot) KFAC_INLINE {
        const int s1 = slot - (r0 + 1), s2 = s1 - (r1 + 1);
        const int r = s1 < 0 ? r0 : s2 < 0 ? r1 : r2, c = s1 < 0 ? slot : s2 < 0 ? s1 : s2;
        if (slot < 11 || c <= r) f(r, c, D[slot]);
    });
}
// Where a lane's four values of 16 x 16 block (r, c) lie in the 32 x 32 block (r / 2, c / 2) in register order (WsView::tile).
__device__ __forceinline__ int sub_block_at(int r, int c, int lane) {
    return (2 * (r & 1) + (lane >> 5)) * 256 + (((lane >> 4) & 1) * 32 + (c & 1) * 16 + (lane & 15)) * 4;
}

// identity beyond nb
__device__ __forceinline__ void pivot_border(PivotBlocks& D, int wave, int nb) {
    const int lane = threadIdx.x & 63;
    each_block(wave, D, [&](int r, int c, v4f& b) KFAC_INLINE {
        const int col = c * PSB + (lane & 15), row = r * PSB + 4 * (lane >> 4);
        auto at = [&](int i, float x) KFAC_INLINE { return row + i < nb && col < nb ? x : row + i == col ? 1.f : 0.f; };
        b = v4f{at(0, b.x), at(1, b.y), at(2, b.z), at(3, b.w)};
    });
}

// Between the rounds of the sweep: everybody's LDS accesses are done.
__device__ __forceinline__ void sweep_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// An owner's part of the sweep.  What the next round needs (columns / rows j + 1, the "strip", and diagonal sub-block j + 2) is brought
// up to date first and handed over; the other blocks follow after the barrier, beside the next round's reads and the inversion of
// wavefront 1, which sets the pace.
// (lds and what is derived from it without __restrict__: what is written through one of them is read through another, also by other wavefronts.)
template <int RL>
__device__ __forceinline__ void sweep_rows(PivotBlocks& blocks, int nsb, float* lds) {
    PivotBlocks D;                                         // (a copy: the compiler would let the owners' branches share accesses, by address)
    static_for<PIV_BLOCKS>([&](auto s) KFAC_INLINE { D[s] = blocks[s]; });
    constexpr int NR = piv_rows(RL), LAST = piv_row(RL, 0);              // (the first row is the longest)
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    float* nat = lds + l16 * PLD + 4 * lq;                               // (l16, 4 lq ..) and (4 lq .., l16) of a panel's 16-row block
    float* turned = lds + 4 * lq * PLD + l16;
    float* diag = lds + PIV_DG + lane * 4;
    constexpr int ROWS = PSB * PLD, PANEL = NB * PLD;
    auto put_turned = [&](int at, const v4f& x) KFAC_INLINE {
        turned[at] = x.x; turned[at + PLD] = x.y; turned[at + 2 * PLD] = x.z; turned[at + 3 * PLD] = x.w;
    };
    v4f T[NR], u[LAST + 1], own[NR], p;
    auto update = [&](auto x, auto c) KFAC_INLINE {        // one 16 x 16 block (T: negated)
        constexpr int at = piv_slot(RL, x) + c, cc = c;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) D[at] = __builtin_amdgcn_mfma_f32_16x16x4f32(T[x][kk], u[cc][kk], D[at], 0, 0, 0);
    };
    static_for<NR>([&](auto x) KFAC_INLINE {
        constexpr int r = piv_row(RL, x), at = piv_slot(RL, x);
        if constexpr (r > 0) put_turned(PIV_US + r * ROWS, D[at]);
        if constexpr (r < 2) *(v4f*)&diag[r * (PSB * PSB)] = D[at + r];
    });
    sweep_barrier();
    sweep_barrier();                                       // wavefront 1 has inverted the first diagonal sub-block
    static_for<NB / PSB + 1>([&](auto round) KFAC_INLINE {
        constexpr int j = round, US = PIV_US + (j & 1) * PANEL, TS = PIV_TS + (j & 1) * PANEL, USN = PIV_US + (~j & 1) * PANEL;
        if (j < nsb) {                                     // (uniform)
            p = *(const v4f*)&nat[PIV_PS + (j & 1) * ROWS];
            static_for<NR>([&](auto x) KFAC_INLINE { own[x] = *(const v4f*)&nat[US + piv_row(RL, x) * ROWS]; });
        }
        if constexpr (j > 0) {
            if (j - 1 < nsb) {                             // the rest of the round before
                constexpr int k = j - 1, TSK = PIV_TS + (k & 1) * PANEL;
                static_for<NR>([&](auto x) KFAC_INLINE {
                    constexpr int r = piv_row(RL, x), at = piv_slot(RL, x);
                    if constexpr (r == k) {                // row k <- T16^T
                        static_for<r>([&](auto c) KFAC_INLINE { D[at + c] = *(const v4f*)&nat[TSK + c * ROWS]; });
                    } else if constexpr (r > k) {          // column k <- T16
                        const float* from = &turned[TSK + r * ROWS];
                        D[at + k] = v4f{from[0], from[PLD], from[2 * PLD], from[3 * PLD]};
                    }
                });
                static_for<NR>([&](auto x) KFAC_INLINE {
                    constexpr int r = piv_row(RL, x);
                    static_for<r + 1>([&](auto c) KFAC_INLINE {
                        if constexpr (r != k && r != j && c != k && c != j && !(c == r && r == k + 2)) update(x, c);
                    });
                });
            }
        }
        if (j < nsb) {
            if constexpr (j < NB / PSB) {
                static_for<LAST + 1>([&](auto c) KFAC_INLINE { u[c] = *(const v4f*)&nat[US + c * ROWS]; });
                // T16 as its transpose P16 . U16^T with v_mfma_f32_16x16x4_f32 (lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]
                // and receives C[4 (l / 16) + i][l % 16], i < 4), the contraction index in the order 4 (l / 16) + kk, so that operands
                // and result are four neighbours of one row: the result is the update's operand.
                static_for<NR>([&](auto x) KFAC_INLINE { T[x] = v4f{0.f, 0.f, 0.f, 0.f}; });
                static_for<4>([&](auto kk) KFAC_INLINE {
                    static_for<NR>([&](auto x) KFAC_INLINE {
                        if constexpr (piv_row(RL, x) != j) T[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[(int)kk], own[x][(int)kk], T[x], 0, 0, 0);
                    });
                });
                static_for<NR>([&](auto x) KFAC_INLINE {
                    constexpr int r = piv_row(RL, x), at = piv_slot(RL, x);
                    if constexpr (r == j) {
                        D[at + r] = -p;
                    } else {
                        *(v4f*)&nat[TS + r * ROWS] = T[x];
                        if constexpr (r == j + 1) put_turned(USN + j * ROWS, T[x]);      // (block (j + 1, j) of the strip)
                        T[x] = -T[x];
                    }
                });
                // the strip: blocks (r, j + 1), r > j + 1, and (j + 1, c), c < j; the diagonal sub-block j + 2.  (The one of j + 1 is
                // wavefront 1's: here it is not needed any more.  Behind the last sub-block there is only padding, which is left out where there is
                // one: up to 16 columns 10.9 to 11.2 us, now 10.7 to 11.0; asked in every round it took registers, 2,049 columns 465 and 479.)
                if (j > 0 || nsb > 1) {                    // (uniform)
                    static_for<NR>([&](auto x) KFAC_INLINE {
                        constexpr int r = piv_row(RL, x);
                        if constexpr (r > j + 1) {
                            update(x, Int<j + 1>());
                            if constexpr (r == j + 2) update(x, Int<r>());
                        } else if constexpr (r == j + 1) {
                            static_for<j>([&](auto c) KFAC_INLINE { update(x, c); });
                        }
                    });
                    static_for<NR>([&](auto x) KFAC_INLINE {
                        constexpr int r = piv_row(RL, x), at = piv_slot(RL, x);
                        if constexpr (r > j + 1) {
                            put_turned(USN + r * ROWS, D[at + j + 1]);
                            if constexpr (r == j + 2) *(v4f*)&diag[(r & 1) * (PSB * PSB)] = D[at + r];
                        } else if constexpr (r == j + 1) {
                            static_for<j>([&](auto c) KFAC_INLINE { *(v4f*)&nat[USN + c * ROWS] = D[at + c]; });
                        }
                    });
                }
                sweep_barrier();
            }
        }
    });
    static_for<PIV_BLOCKS>([&](auto s) KFAC_INLINE { blocks[s] = D[s]; });
}

// The symmetric sweep of D in 16-wide sub-blocks (see above); lds: PIV_LDS_FLOATS floats, free on entry.  Returns (to every
// thread) the 1-based index inside the block of the first non-positive pivot, or 0.  Ends with a barrier.
__device__ __forceinline__ int pivot_sweep(PivotBlocks& D, int wave, int nb, float* lds) {
    int* bad = (int*)(lds + PIV_BAD);
    const int nsb = (nb + PSB - 1) / PSB;
    if (wave == 1) {
        const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
        sweep_barrier();                                       // the first U16 and the diagonal sub-blocks are there
        v4f N = -*(const v4f*)&lds[PIV_DG + lane * 4];
        int first_bad = invert16_wave(N, lds + PIV_PS);
        sweep_barrier();
#pragma unroll 1
        for (int n = 1; n < nsb; ++n) {                        // diagonal sub-block n -= T16 . U16^T, and its inverse
            // (N: the inverse of the sub-block before; T16 as in sweep_rows, for these 16 rows, stays in registers; the sum is
            // formed by itself and added at once: most of it cancels)
            const v4f u = *(const v4f*)&lds[PIV_US + ((n - 1) & 1) * (NB * PLD) + (n * PSB + l16) * PLD + 4 * lq];
            const v4f old = *(const v4f*)&lds[PIV_DG + (n & 1) * (PSB * PSB) + lane * 4];
            v4f tt = {0.f, 0.f, 0.f, 0.f}, sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) tt = __builtin_amdgcn_mfma_f32_16x16x4f32(N[kk], u[kk], tt, 0, 0, 0);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) sum = __builtin_amdgcn_mfma_f32_16x16x4f32(tt[kk], u[kk], sum, 0, 0, 0);
            // the accumulator layout holds (row 4 lq + i, column l16): by symmetry element (l16, 4 lq + i)
            N = sum - old;
            const int f = invert16_wave(N, lds + PIV_PS + (n & 1) * (PSB * PLD));
            first_bad = f != 0 && first_bad == 0 ? n * PSB + f : first_bad;
            sweep_barrier();
        }
        if (lane == 0) *bad = first_bad;
        sweep_barrier();
    } else {
        with_role(wave, [&](auto role) KFAC_INLINE { sweep_rows<role>(D, nsb, lds); });
    }
    const int f = *bad;
    sweep_barrier();                                           // everybody has read what there is to read: the memory may be reused
    return f;
}

// D holds -P up to rounding asymmetry on and below the diagonal.  The working copy gets -P; on the matrix's last step the
// caller's output gets +P (the final sign flip; lower triangle taken as the truth, so that it is exactly symmetric) instead.
// The workspace gets +P for the panel product, all of it.
__device__ __forceinline__ void pivot_write(PivotBlocks& D, int wave, float* tri, const Item& it,
                                            const WsView& ws, int k0, int nb, bool last, bool from_S) {
    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, lq = lane >> 4;
    const int d = it.dim;
    gfloat* P = ws.P(k0 / NB);
    if (!last) {                                           // (then the block is full)
        // A full block inside the sweep (the look-ahead pivot's usual case) goes out as it lies in the registers: 16 lanes hold 16
        // consecutive floats of a row, and a lane four consecutive floats of the mirror image's.
        gfloat* tile = ws.tile(k0 / NB, k0 / NB);
        each_block(wave, D, [&](int r, int c, const v4f& b) KFAC_INLINE {
            *(KFAC_AS1 v4f*)(tile_block(tile, r >> 1, c >> 1) + sub_block_at(r, c, lane)) = b;
            *(KFAC_AS1 v4f*)&P[(c * PSB + l16) * NB + r * PSB + 4 * lq] = -b;
            if (r == c) return;                            // a block on the diagonal is its own mirror image
#pragma unroll
            for (int i = 0; i < 4; ++i) P[(r * PSB + 4 * lq + i) * NB + c * PSB + l16] = -b[i];
        });
        return;
    }
    each_block(wave, D, [&](int r, int c, const v4f& b) KFAC_INLINE {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = r * PSB + 4 * lq + i, col = c * PSB + l16;
            if (row >= col) tri[tri_at(row, col)] = b[i];
        }
    });
    __syncthreads();
    // thread = four consecutive columns of one row, 8 rows per pass: 16-byte stores (the working copy and the P
    // buffer are 16-byte aligned; the caller's output need not be)
    const int c4 = (t & 31) * 4, r0 = t >> 5;
#pragma unroll 4
    for (int p = 0; p < 16; ++p) {
        const int row = r0 + 8 * p;
        if (row >= nb || c4 >= nb) continue;
        v4f x;
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = tri[tri_sym(row, min(c4 + i, nb - 1))];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (c4 + i < nb) it.Minv[(size_t)(k0 + row) * d + k0 + c4 + i] = -x[i];
        if (!from_S) *(KFAC_AS1 v4f*)&P[row * NB + c4] = -x;    // (columns beyond a ragged block are never read)
    }
}

// The first pivot block of a matrix, S + lambda I; the only one of a single-block matrix, whose output this writes.
__device__ __forceinline__ void begin_pivot(const Item& it, float* lds) {
    const int d = it.dim, nb = min(NB, d);
    const bool single = d <= NB;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const WsView ws = ws_view(it.ws, d);
    // straight into the accumulators, of the lower triangle; indices clamped, not guarded, so that all loads go out together
    PivotBlocks D;
    const int l16 = lane & 15, l4 = 4 * (lane >> 4);
    each_block(wave, D, [&](int r, int c, v4f& b) KFAC_INLINE {
        auto at = [&](int i) KFAC_INLINE {
            const int row = min(r * PSB + l4 + i, nb - 1), col = min(c * PSB + l16, nb - 1);
            return it.S[(size_t)max(row, col) * d + min(row, col)];
        };
        b = v4f{at(0), at(1), at(2), at(3)};
    });
    const v4f lambda = {l4 == l16 ? it.damping : 0.f, l4 + 1 == l16 ? it.damping : 0.f, l4 + 2 == l16 ? it.damping : 0.f,
                        l4 + 3 == l16 ? it.damping : 0.f};
    each_block(wave, D, [&](int r, int c, v4f& b) KFAC_INLINE {
        if (r == c) b += lambda;
    });
    if (nb < NB) pivot_border(D, wave, nb);
    const int f = pivot_sweep(D, wave, nb, lds);
    if (t == 0 && it.info) *it.info = f;                 // (later pivots: step_pivot)
    pivot_write(D, wave, lds, it, ws, 0, nb, single, single);
}

// A quarter (32 rows) of tile (I, J) of the working copy: W(lower) = S(lower) + lambda I.  Tiles on the diagonal get both
// triangles (of S's lower one): the pivot code works on whole 32 x 32 diagonal blocks, which the updates keep whole.
__device__ __forceinline__ void begin_tile(const Item& it, int I, int J, int quarter) {
    const int d = it.dim;
    const gfloat* __restrict__ S = it.S;
    const int lane = threadIdx.x & 63, cb = threadIdx.x >> 6;
    const int c = cb * 32 + (lane & 31), r0 = quarter * 32 + 4 * (lane >> 5);    // inside the tile
    const int col = J * NB + c;
    v16f v;
#pragma unroll
    for (int r = 0; r < 16; ++r) {                       // loads only: arithmetic on a guarded load would make the
        const int row = I * NB + r0 + (r >> 2) * 8 + (r & 3);            // compiler wait for each load in turn
        v[r] = row < d && col < d ? S[(size_t)max(row, col) * d + min(row, col)] : 0.f;
    }
    if (I == J) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (r0 + (r >> 2) * 8 + (r & 3) == c) v[r] += it.damping;
    }
    store_block(tile_block(ws_view(it.ws, d).tile(I, J), quarter, cb), v);
}

// Half a slab (64 rows) of panel `step`: the scale and the fp16 pieces of U that the tile products read, and U itself.  v[p]: columns
// c4 .. c4 + 3 of row rr + 8 p, c4 = 4 (t % 32), rr = t / 32.
__device__ __forceinline__ void put_panel(const WsView& ws, int step, int slab, int half, const v4f (&v)[8], float* __restrict__ red) {
    const int t = threadIdx.x, c4 = (t & 31) * 4, rr = t >> 5, q = step % NBUF;
    gfloat* __restrict__ Uc = ws.U(q) + (size_t)(slab * NB + half * PH) * NB;
    float um = 0.f;
#pragma unroll
    for (int p = 0; p < 8; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) um = fmaxf(um, fabsf(v[p][i]));
    um = block_absmax(um, red);
    const float su = panel_scale(um);
    if (t == 0) ws.scaleU(q, 2 * slab + half) = su;
    KFAC_AS1 unsigned char* uh = ws.UH(q) + (size_t)slab * PRE_SLAB;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        *(KFAC_AS1 v4f*)&Uc[(size_t)(rr + 8 * p) * NB + c4] = v[p];
        store_split4_h2(uh, uh + ws.plane, half * PH + rr + 8 * p, c4, v[p] * su);
    }
}

// Panel 0, straight from the factor.
__device__ __forceinline__ void begin_panel(const Item& it, int slab, int half, float* __restrict__ red) {
    const int d = it.dim, t = threadIdx.x, c4 = (t & 31) * 4, r0 = slab * NB + half * PH + (t >> 5);
    v4f v[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) {                        // (rows clamped, not guarded: all loads go out together)
        const int row = r0 + 8 * p;
        v[p] = *(const KFAC_AS1 v4f_a4*)(it.S + (size_t)min(row, d - 1) * d + c4);
    }
#pragma unroll
    for (int p = 0; p < 8; ++p)
        if (r0 + 8 * p >= d) v[p] = v4f{0.f, 0.f, 0.f, 0.f};
    put_panel(ws_view(it.ws, d), 0, slab, half, v, red);
}

// The working copy's workgroups of a matrix of n blocks: the half slabs of panel 0, then the quarter tiles of the rest.
static inline __host__ __device__ int begin_workgroups(int n) { return 2 * (n - 1) + 4 * (n * (n - 1) / 2); }
__device__ __forceinline__ void begin_tile_of(const Batch& b, int wg, float* __restrict__ red) {
    int m, local;
    locate(b, wg, m, local);
    const Item it = get_item(b, m);
    const int panel = 2 * (nblk_of(it.dim) - 1);
    if (local < panel) {
        begin_panel(it, 1 + (local >> 1), local & 1, red);
        return;
    }
    local -= panel;
    int I, J;
    tri_decode(local >> 2, I, J);
    begin_tile(it, I + 1, J + 1, local & 3);
}

// Start of every matrix of the batch: its first pivot block and, in the workgroups after the pivots', the damped working copy
// (of matrices with more than one block; the tile of the pivot block is the pivot's to write).  The copies are done before
// the pivots are; in a launch before the pivots' they took 15 us of every inversion's chain.
__global__ __launch_bounds__(256) void inv_begin_kernel(Batch b) {
    __shared__ __attribute__((aligned(16))) float lds[PIV_LDS_FLOATS];
    if ((int)blockIdx.x < b.count) {
        __builtin_amdgcn_s_setprio(3);
        begin_pivot(get_item(b, blockIdx.x), lds);
        return;
    }
    begin_tile_of(b, blockIdx.x - b.count, lds);
}

// The working copies alone, for batches whose copies do not fit the chip beside the pivots: these workgroups need a tenth of
// the pivot's registers and no LDS, and find room between those of other streams (a network's step at batch 32, whose
// factor builds run beside: 5.87 ms, with the copies in the pivots' launch 6.07 ms).
__global__ __launch_bounds__(256) void inv_init_kernel(Batch b) {
    __shared__ float red[4];
    begin_tile_of(b, blockIdx.x, red);
}
constexpr int BEGIN_TOGETHER = 768;      // workgroups; a CU runs one at a time of inv_begin_kernel, which has the pivot's registers

// acc = T . U^T of a matrix's last step, fp32, with both operand slabs (128 rows x nb floats, row stride 128, zero beyond nb)
// streamed through a 3-stage LDS ring by global_load_lds_dwordx4 (lane i's 16 bytes land at block base + 16 i), so
// no registers are spent on staging and one barrier per 16-wide K-slab suffices.  Inside a 1 KB block (16 rows x 4
// chunks of 4 floats) chunk c of row r sits in slot 4 r + (c ^ ((r >> 1) & 3)): the MFMA operand reads (one float4
// per lane, 32 consecutive rows per half-wave) are then bank-conflict free.
constexpr int UK = 16;                    // K-slab
constexpr int UNS = 3;                    // ring stages
constexpr int UPANEL = 8 * 1024;          // bytes per operand panel per stage
constexpr int USTAGE = 2 * UPANEL;
static_assert(UNS * USTAGE <= UPD_LDS_BYTES && PRE_NS * PRE_STAGE <= UPD_LDS_BYTES && HALF_NS * HALF_STAGE <= UPD_LDS_BYTES &&
              GEMM_LDS_FLOATS * 4 <= UPD_LDS_BYTES && PIV_LDS_FLOATS * 4 <= UPD_LDS_BYTES, "all uses share the kernel's LDS");

#define KFAC_LDS_READ128(dst, addr, off) \
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off))

__device__ __forceinline__ void product_f32(const gfloat* __restrict__ T, const gfloat* __restrict__ U, int nb, bool dead, float* __restrict__ lds,
                                            TileAcc& acc) {
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int lm = lane & 31, h = lane >> 5;
    lds_byte* l0 = (lds_byte*)lds;

    // ---- producer: wavefronts 0,1 stream T_I, wavefronts 2,3 stream U_J; four 1 KB blocks each per stage ----
    const int pan = wave >> 1;
    const int drow = lane >> 2, dchunk = (lane & 3) ^ ((lane >> 3) & 3);
    const gfloat* src0 = (pan == 0 ? T : U) + (size_t)drow * NB + 4 * dchunk;
    const int nst = (nb + UK - 1) / UK;
    auto issue = [&](int s, int buf) {
        const int sc = s < nst ? s : nst - 1;              // past the end: re-read the last slab (never consumed)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int b = (wave & 1) + 2 * j;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src0 + (size_t)(16 * b) * NB + sc * UK),
                                             (__attribute__((address_space(3))) void*)(l0 + buf * USTAGE + pan * UPANEL + b * 1024),
                                             16, 0, 0);
        }
    };

    // ---- consumer: per-lane LDS byte addresses of the float4 holding k = 8 s2 + 4 h .. +3 of its row ----
    unsigned a_addr[2][2], b_addr[2][2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const int ma = wm * 64 + q * 32 + lm, mb_ = wn * 64 + q * 32 + lm;
            const int ch = 2 * s2 + h;
            a_addr[q][s2] = (unsigned)((ma >> 4) * 1024 + (4 * (ma & 15) + (ch ^ (((ma & 15) >> 1) & 3))) * 16);
            b_addr[q][s2] = (unsigned)(UPANEL + (mb_ >> 4) * 1024 + (4 * (mb_ & 15) + (ch ^ (((mb_ & 15) >> 1) & 3))) * 16);
        }

#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nbk = 0; nbk < 2; ++nbk)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc.c[mb][nbk][r] = 0.f;
    issue(0, 0);
    issue(1, 1);
    for (int it = 0; it < nst; it += UNS) {
#pragma unroll
        for (int bi = 0; bi < UNS; ++bi) {
            const int s = it + bi;
            if (s >= nst) break;                                            // uniform
            asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");   // slab s landed (everybody's part)
            issue(s + 2, (bi + 2) % UNS);                                    // refill the slot slab s-1 vacated
            if (!dead) {
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    v4f a[2], bb[2];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        KFAC_LDS_READ128(a[q], a_addr[q][s2], bi * USTAGE);
                        KFAC_LDS_READ128(bb[q], b_addr[q][s2], bi * USTAGE);
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(bb[0]), "+v"(bb[1]));
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                            for (int nbk = 0; nbk < 2; ++nbk)
                                acc.c[mb][nbk] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mb][i], bb[nbk][i], acc.c[mb][nbk], 0, 0, 0);
                }
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");            // ring idle: the LDS may be reused
}

// Where a tile's old values come from.
struct OldSrc {
    int kind;                // OLD_W, OLD_T, OLD_T_TURNED
    const gfloat* base;      // the tile, or the first of the slab's rows
};

// Old values of this wavefront's quadrant, in the accumulators' order.  `dead`: the quadrant above the diagonal of a diagonal tile.
__device__ __forceinline__ void load_old(const OldSrc& o, bool dead, TileAcc& acc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nbk = 0; nbk < 2; ++nbk) {
            if (dead) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc.c[mb][nbk][r] = 0.f;
            } else if (o.kind == OLD_W) {                 // (uniform)
                load_block(o.base + ((2 * wm + mb) * 4 + 2 * wn + nbk) * 1024, acc.c[mb][nbk]);
            } else if (o.kind == OLD_T) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc.c[mb][nbk][r] = o.base[acc_row(wm, mb, r, lane) * NB + acc_col(wn, nbk, lane)];
            } else {
#pragma unroll
                for (int r = 0; r < 16; r += 4) {
                    const v4f x = *(const KFAC_AS1 v4f*)&o.base[acc_col(wn, nbk, lane) * NB + acc_row(wm, mb, r, lane)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc.c[mb][nbk][r + i] = x[i];
                }
            }
        }
}

// The products of a tile, of all steps but the matrix's last one: new = old - A0 B0^T - A1 B1^T - ... (one product per pending
// step, in step order).  Only a matrix's last block can be ragged and the step that eliminates it is its last, so here the pivot
// blocks are full (K = 128 per product).  The products run on the fp16 matrix cores with both operands scaled per
// half slab and split two ways (gemm_split.h): the accumulators start as the tile's old values, the negated products are added,
// and the result is stored from the registers: nothing is staged in LDS.
constexpr int MAXRUN = GM;               // a tile owes at most one whole group (the group before, or its own so far)
static_assert(HALF_MAXN == GM + 1, "a half slab owes at most the group before and one step (chain_from)");
typedef SplitRun<MAXRUN> PanelRun;

// The products of tile (I, J) with the panels of the n consecutive steps first_step .. first_step + n - 1 (buffer =
// step mod NBUF).
__device__ __forceinline__ PanelRun panel_run(const WsView& ws, int first_step, int n, int I, int J) {
    // (a wavefront's quadrant is one half slab by one half slab: one scale)
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1;
    PanelRun r;
    r.a_hi = ws.TH(0) + (size_t)I * PRE_SLAB;
    r.b_hi = ws.UH(0) + (size_t)J * PRE_SLAB;
    r.plane = ws.plane;
    r.stride = ws.stride * sizeof(float);
    r.first = first_step % NBUF;
    r.nbuf = NBUF;
    r.n = n;
#pragma unroll
    for (int q = 0; q < MAXRUN; ++q) {
        const int b = (first_step + q) % NBUF;
        r.scale[q] = ws.scaleT(b, 2 * I + wm) * ws.scaleU(b, 2 * J + wn);
    }
    return r;
}

// T = U . P for half a slab (64 rows): the fp32 panel and the scaled, negated fp16 pieces that the tile products read, with their
// scale (returned).  Half slabs: twice the workgroups for a link of the chain that leaves most CUs idle, and half the time in every
// phase.  The product runs on the bf16 matrix cores with both operands split three ways (panel_product).  pb: P's values
// (panel_fetch_b).  Ends with the LDS free and T's stores on their way.
constexpr int PANEL_RLD = NB + 4;          // LDS row stride of the stage, read back four columns at a time
static_assert(UPD_LDS_BYTES >= PANEL_B_LDS && UPD_LDS_BYTES >= PH * PANEL_RLD * 4, "one buffer serves all uses");

// (accumulators of a 64 x 128 half slab: wavefront (wm, wn) holds rows 32 wm .. of columns 64 wn .., as two MFMA blocks)
__device__ __forceinline__ int half_row(int wm, int r, int lane) { return wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3); }

__device__ __forceinline__ void half_stage(const v16f (&acc)[2], float* __restrict__ lds) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int nbk = 0; nbk < 2; ++nbk)
#pragma unroll
        for (int r = 0; r < 16; ++r) lds[half_row(wm, r, lane) * PANEL_RLD + acc_col(wn, nbk, lane)] = acc[nbk][r];
}

__device__ __forceinline__ float slab_T(const WsView& ws, int step, int slab, int half, const v4f (&pb)[8][2], float* __restrict__ lds,
                                        float* __restrict__ red) {
    const int t = threadIdx.x, q = step % NBUF, r0 = slab * NB + half * PH;
    const int c4 = (t & 31) * 4, rr = t >> 5;
    v16f acc[2];
    panel_product(ws.U(q) + (size_t)r0 * NB, pb, (unsigned char*)lds, acc);
    float tm = 0.f;
#pragma unroll
    for (int nbk = 0; nbk < 2; ++nbk)
#pragma unroll
        for (int r = 0; r < 16; ++r) tm = fmaxf(tm, fabsf(acc[nbk][r]));
    tm = block_absmax(tm, red);                          // (its barriers also separate the product's LDS use from this one)
    const float st = panel_scale(tm);
    if (t == 0) ws.scaleT(q, 2 * slab + half) = st;
    half_stage(acc, lds);
    __syncthreads();
    gfloat* __restrict__ Tc = ws.T(q) + (size_t)r0 * NB;
    KFAC_AS1 unsigned char* th = ws.TH(q) + (size_t)slab * PRE_SLAB;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const int row = rr + 8 * p;
        const v4f x = *(const v4f*)&lds[row * PANEL_RLD + c4];
        *(KFAC_AS1 v4f*)&Tc[(size_t)row * NB + c4] = x;       // (zeros beyond the matrix, as in U)
        store_split4_h2(th, th + ws.plane, half * PH + row, c4, x * -st);
    }
    __threadfence_block();
    __syncthreads();                                     // T is visible to the workgroup; the stage is free
    return st;
}

// The operands of half slab (I, half) times slab J for the n consecutive steps first .. first + n - 1, the last of them `step`, whose
// T this workgroup has just formed (st: its scale).
__device__ __forceinline__ HalfRun half_run(const WsView& ws, int first, int step, int I, int half, int J, float st) {
    const int wn = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) & 1;
    HalfRun r;
    r.a_hi = ws.TH(0) + (size_t)I * PRE_SLAB + half * (PRE_BLOCK / 2);
    r.b_hi = ws.UH(0) + (size_t)J * PRE_SLAB;
    r.plane = ws.plane;
    r.stride = ws.stride * sizeof(float);
    r.first = first % NBUF;
    r.nbuf = NBUF;
    r.n = step - first + 1;
#pragma unroll
    for (int q = 0; q < HALF_MAXN; ++q) {
        const int b = (first + q) % NBUF;
        r.scale[q] = first + q < step ? ws.scaleT(b, 2 * I + half) * ws.scaleU(b, 2 * J + wn) : st * ws.scaleU(b, 2 * J + wn);
    }
    return r;
}

// One half slab of step k: T, then the half slab of panel k + 1 (and, for the block after that, half of its diagonal tile).
__device__ __forceinline__ void step_slab(const Item& it, int k, int I, int half, float* __restrict__ lds, float* __restrict__ red) {
    const int d = it.dim, c1 = k + 1;
    const WsView ws = ws_view(it.ws, d);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int lm = lane & 31, h = lane >> 5;
    v4f pb[8][2];
    v16f acc[2];
    if (I == k) {
        // block row k + 1 left of the diagonal, in block column k: T_(k+1) transposed = P U_(k+1)^T
        panel_fetch_b(ws.U(k % NBUF) + (size_t)c1 * NB * NB, pb);
        panel_product(ws.P(k) + half * PH * NB, pb, (unsigned char*)lds, acc);
        __syncthreads();
    } else {
        panel_fetch_b(ws.P(k), pb);
        const float st = slab_T(ws, k, I, half, pb, lds, red);
        if (I == c1) return;                             // (the tile itself is the look-ahead pivot's)
        // Old values of tile (I, k + 1) in the accumulators' order.  Left of the diagonal the tile is stored as (k + 1, I); a block
        // that was eliminated since the working copy was last up to date left it in that step's T.
        int first = chain_from(c1);
        const int ab = 2 * half + wm;                    // this wavefront's block of the slab's rows
        if (I > c1) {
#pragma unroll
            for (int nbk = 0; nbk < 2; ++nbk) load_block(tile_block(ws.tile(I, c1), ab, 2 * wn + nbk), acc[nbk]);
        } else if (I >= first) {                         // (first <= I < k)
            first = I + 1;
            const gfloat* src = ws.T(I % NBUF) + (size_t)(c1 * NB + wn * 64 + lm) * NB + ab * 32 + 4 * h;
#pragma unroll
            for (int nbk = 0; nbk < 2; ++nbk)
#pragma unroll
                for (int r = 0; r < 16; r += 4) {
                    const v4f x = *(const KFAC_AS1 v4f*)(src + nbk * (32 * NB) + 2 * r);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[nbk][r + i] = x[i];
                }
        } else {
            const gfloat* tile = ws.tile(c1, I) + (lm >> 3) * 256 + ((lm >> 2) & 1) * 128 + (lm & 3) + 16 * h;
#pragma unroll
            for (int nbk = 0; nbk < 2; ++nbk)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nbk][r] = tile[((2 * wn + nbk) * 4 + ab) * 1024 + (r >> 2) * 32 + (r & 3) * 4];
        }
        const float back = half_mma_presplit(half_run(ws, first, k, I, half, c1, st), (unsigned char*)lds, acc);
#pragma unroll
        for (int nbk = 0; nbk < 2; ++nbk) acc[nbk] *= back;
        if (I == k + 2) {
            half_stage(acc, lds);
            __syncthreads();
            v4f v[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) v[p] = *(const v4f*)&lds[((t >> 5) + 8 * p) * PANEL_RLD + (t & 31) * 4];
            put_panel(ws, c1, I, half, v, red);
            // the diagonal tile of block k + 2: steps k - 1 and k
            gfloat* tile = ws.tile(I, I);
#pragma unroll
            for (int nbk = 0; nbk < 2; ++nbk) load_block(tile_block(tile, ab, 2 * wn + nbk), acc[nbk]);
            const float back2 = half_mma_presplit(half_run(ws, max(0, k - 1), k, I, half, I, st), (unsigned char*)lds, acc);
#pragma unroll
            for (int nbk = 0; nbk < 2; ++nbk) store_block(tile_block(tile, ab, 2 * wn + nbk), acc[nbk] * back2);
            return;
        }
    }
    half_stage(acc, lds);
    __syncthreads();
    v4f v[8];
#pragma unroll
    for (int p = 0; p < 8; ++p) v[p] = *(const v4f*)&lds[((t >> 5) + 8 * p) * PANEL_RLD + (t & 31) * 4];
    put_panel(ws, c1, I, half, v, red);
}

// One half slab of the last step's panel.  Ragged pivot block: fp32 matrix cores, a workgroup per slab.
__device__ __forceinline__ void last_slab(const Item& it, int k, int I, int half, float* __restrict__ lds, float* __restrict__ red) {
    const int d = it.dim, nb = d - k * NB, q = k % NBUF;
    const WsView ws = ws_view(it.ws, d);
    if (nb == NB) {
        v4f pb[8][2];
        panel_fetch_b(ws.P(k), pb);
        slab_T(ws, k, I, half, pb, lds, red);
        return;
    }
    if (half == 1) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    gfloat* __restrict__ Tc = ws.T(q) + (size_t)I * NB * NB;
    TileAcc acc;
    tile_mma_nt(ws.U(q) + (size_t)I * NB * NB, NB, NB, ws.P(k), NB, nb, nb, lds, acc);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nbk = 0; nbk < 2; ++nbk)
#pragma unroll
            for (int r = 0; r < 16; ++r) {                // (the output's products stream whole 16-float slices of T: zeros beyond nb)
                const int row = acc_row(wm, mb, r, lane), col = acc_col(wn, nbk, lane);
                Tc[(size_t)row * NB + col] = col < nb ? acc.c[mb][nbk][r] : 0.f;
            }
}

// Look-ahead: the diagonal tile that is the next step's pivot block is updated by a workgroup of its own, which keeps the new
// values in registers and inverts the block at once.  It is the launch's longest workgroup, so the update is formed from what the
// launch starts with, without waiting for the slab's T to be written: T^T = P U^T, every wavefront for 32 rows of T, leaves the
// matrix cores in registers that serve, scaled and split into fp16 pieces, as the operand of T U^T (the contraction index in the
// order the accumulators hold it; U's pieces are read in the same order).  U's pieces come by LDS copies that start before the
// first product, and, as far as the LDS does not hold them yet, through registers that the first product no longer needs.  D: acc (blocks on and below the diagonal), from W's tile.
// Taken from the slab's T as the other workgroups write it, two half slabs one after the other: 19 us until the sweep begins, and 26
// with a tile's workgroup on the same CU.
constexpr int PUP_RING = PANEL_B_LDS;                    // LDS: P's pieces (panel_stash), then three slices of U's; later six
static_assert(PUP_RING + 3 * 2 * PRE_BLOCK <= UPD_LDS_BYTES && 10 * 4096 <= UPD_LDS_BYTES, "the kernel's LDS");

__device__ __forceinline__ void pivot_update(const WsView& ws, int step, unsigned char* lds, PivotBlocks& D) {
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const int kn = step + 1, q = step % NBUF;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), lm = lane & 31, h = lane >> 5;
    lds_byte* l0 = (lds_byte*)lds;
    const gfloat* P = ws.P(step);
    const KFAC_AS1 unsigned char* uh = ws.UH(q) + (size_t)kn * PRE_SLAB + lane * 16;
    auto copy_slice = [&](int s, int at) {               // both planes of slice s to LDS offset `at`: 8 KB, two copies a wavefront
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int kb = 2 * wave + j;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(uh + (kb >= 4 ? ws.plane : 0) + s * PRE_BLOCK + (kb & 3) * 1024),
                                             (__attribute__((address_space(3))) void*)(l0 + at + kb * 1024), 16, 0, 0);
        }
    };
    const KFAC_AS1 unsigned char* ur = ws.UH(q) + (size_t)kn * PRE_SLAB + (wave >> 1) * ws.plane + (wave & 1) * 2048 + lane * 16;
    auto fetch_slice = [&](int s, v4f (&x)[2]) {         // the same by way of registers
#pragma unroll
        for (int j = 0; j < 2; ++j) x[j] = *(const KFAC_AS1 v4f*)(ur + s * PRE_BLOCK + j * 1024);
    };
    auto put_slice = [&](int at, const v4f (&x)[2]) {
#pragma unroll
        for (int j = 0; j < 2; ++j) *(v4f*)(lds + at + (2 * wave + j) * 1024 + lane * 16) = x[j];
    };
    // ---- T^T = P U^T: block kb holds rows (of P, the contraction index of the second product) 32 kb .., columns = rows 32 wave .. of T
    constexpr int AHEAD = 4;                             // slices of P in flight
    v4f pb[AHEAD][2], xa[3][2];
    panel_fetch_slice(P, 0, pb[0]);
    const gfloat* urow = ws.U(q) + ((size_t)kn * NB + wave * 32 + lm) * NB + 8 * h;
    auto fetch_u = [&](int s, v4f (&x)[2]) {
        x[0] = *(const KFAC_AS1 v4f*)(urow + s * SPLIT_KS);
        x[1] = *(const KFAC_AS1 v4f*)(urow + s * SPLIT_KS + 4);
    };
    fetch_u(0, xa[0]);
#pragma unroll
    for (int s = 1; s < AHEAD; ++s) panel_fetch_slice(P, s, pb[s]);
    fetch_u(1, xa[1]);
#pragma unroll
    for (int s = 0; s < 3; ++s) copy_slice(s, PUP_RING + s * 2 * PRE_BLOCK);
    // the tile's old values, into this XCD's L2: two of its 512 cache lines a thread
    gfloat* wtile = ws.tile(kn, kn);
    const float touch[2] = {wtile[t * 64], wtile[t * 64 + 32]};
    const float su[2] = {ws.scaleU(q, 2 * kn), ws.scaleU(q, 2 * kn + 1)};
    unsigned a_off[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) a_off[kb] = (unsigned)split_plane_offset(kb * 32 + lm, h);
    v16f tt[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) tt[kb][r] = 0.f;
    panel_stash(lds, 0, pb[0]);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        if (s + AHEAD < 8) panel_fetch_slice(P, s + AHEAD, pb[s % AHEAD]);
        if (s + 2 < 8) fetch_u(s + 2, xa[(s + 2) % 3]);
        uint2 lo[3], hi[3];
        uint4 u[3];
        split4<3>(xa[s % 3][0], lo);
        split4<3>(xa[s % 3][1], hi);
#pragma unroll
        for (int e = 0; e < 3; ++e) u[e] = make_uint4(lo[e].x, lo[e].y, hi[e].x, hi[e].y);
        uint4 p[2][3];                                   // (the next block's pieces are on their way beside a block's products)
        auto read_p = [&](int kb) {
#pragma unroll
            for (int e = 0; e < 3; ++e) p[kb & 1][e] = *(const uint4*)(lds + (s & 1) * (3 * SPLIT_PLANE) + e * SPLIT_PLANE + a_off[kb]);
        };
        read_p(0);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            if (kb + 1 < 4) read_p(kb + 1);
            // smallest terms first
#pragma unroll
            for (int order = 2; order >= 0; --order)
#pragma unroll
                for (int pa = 0; pa <= order; ++pa) tt[kb] = mfma16<false>(p[kb & 1][pa], u[order - pa], tt[kb]);
        }
        if (s + 1 < 8) panel_stash(lds, s + 1, pb[(s + 1) % AHEAD]);
        if (s >= 3 && s < 7) fetch_slice(s, pb[(s + 1) % AHEAD]);        // (free from here on)
        __syncthreads();
    }
    fetch_slice(7, xa[0]);
    asm volatile("" :: "v"(touch[0]), "v"(touch[1]));
    // ---- T U^T: row block `wave`, column blocks 0 .. wave
    // (U's first three slices landed before the last of P's: this wavefront's loads return in order; P's pieces are done with)
#pragma unroll
    for (int s = 3; s < 6; ++s) put_slice((s - 3) * 2 * PRE_BLOCK, pb[(s + 1) % AHEAD]);
    float tm = 0.f;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) tm = fmaxf(tm, fabsf(tt[kb][r]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) tm = fmaxf(tm, __shfl_xor(tm, off, 64));
    const float st = panel_scale(tm);
    v16f dd[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) dd[cb][r] = 0.f;
    auto slice = [&](int s, int at) {
        uint2 p0[2], p1[2];
        const v4f x0 = {tt[s >> 1][8 * (s & 1)] * st, tt[s >> 1][8 * (s & 1) + 1] * st, tt[s >> 1][8 * (s & 1) + 2] * st, tt[s >> 1][8 * (s & 1) + 3] * st};
        const v4f x1 = {tt[s >> 1][8 * (s & 1) + 4] * st, tt[s >> 1][8 * (s & 1) + 5] * st, tt[s >> 1][8 * (s & 1) + 6] * st, tt[s >> 1][8 * (s & 1) + 7] * st};
        split4_h2(x0, p0);
        split4_h2(x1, p1);
        const uint4 a[2] = {make_uint4(p0[0].x, p0[0].y, p1[0].x, p1[0].y), make_uint4(p0[1].x, p0[1].y, p1[1].x, p1[1].y)};
        uint4 b[2][2];
        auto read_b = [&](int cb) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const unsigned char* src = lds + at + e * PRE_BLOCK + 8 * h;
                const uint2 x = *(const uint2*)(src + split_plane_offset(cb * 32 + lm, 0)), y = *(const uint2*)(src + split_plane_offset(cb * 32 + lm, 1));
                b[cb & 1][e] = make_uint4(x.x, x.y, y.x, y.y);
            }
        };
        read_b(0);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            if (cb > wave) continue;                     // (uniform)
            if (cb + 1 < 4) read_b(cb + 1);
            dd[cb] = mfma16<true>(a[1], b[cb & 1][0], dd[cb]);
            dd[cb] = mfma16<true>(a[0], b[cb & 1][1], dd[cb]);
            dd[cb] = mfma16<true>(a[0], b[cb & 1][0], dd[cb]);
        }
    };
#pragma unroll
    for (int s = 0; s < 3; ++s) slice(s, PUP_RING + s * 2 * PRE_BLOCK);
    __syncthreads();                                     // slices 3 .. 5 are there, 0 .. 2 are done with
    put_slice(PUP_RING, pb[(6 + 1) % AHEAD]);
    put_slice(PUP_RING + 2 * PRE_BLOCK, xa[0]);
#pragma unroll
    for (int s = 3; s < 6; ++s) slice(s, (s - 3) * 2 * PRE_BLOCK);
    __syncthreads();
#pragma unroll
    for (int s = 6; s < 8; ++s) slice(s, PUP_RING + (s - 6) * 2 * PRE_BLOCK);
    each_block(wave, D, [&](int r, int c, v4f& b) KFAC_INLINE { b = *(const KFAC_AS1 v4f*)(tile_block(wtile, r >> 1, c >> 1) + sub_block_at(r, c, lane)); });
    // ---- to the wavefronts that own the block rows, 32 x 32 block by block in register order
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");          // U's pieces are done with
    float* blocks = (float*)lds;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
        if (cb > wave) continue;
        const float back = 1.0f / (st * su[cb >> 1]);
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            const v4f x = {dd[cb][r] * back, dd[cb][r + 1] * back, dd[cb][r + 2] * back, dd[cb][r + 3] * back};
            *(v4f*)&blocks[(wave * (wave + 1) / 2 + cb) * 1024 + r * 64 + lane * 4] = x;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    each_block(wave, D, [&](int r, int c, v4f& b) KFAC_INLINE {
        const int rb = r >> 1, cb = c >> 1;
        b -= *(const v4f*)&blocks[(rb * (rb + 1) / 2 + cb) * 1024 + sub_block_at(r, c, lane)];
    });
    __syncthreads();
}

__device__ __forceinline__ void step_pivot(const Item& it, int step, float* lds) {
    const int d = it.dim, k0 = (step + 1) * NB, nb = min(NB, d - k0);
    const WsView ws = ws_view(it.ws, d);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    PivotBlocks D;
    pivot_update(ws, step, (unsigned char*)lds, D);
    if (nb < NB) pivot_border(D, wave, nb);              // (uniform)
    const int f = pivot_sweep(D, wave, nb, lds);
    if (threadIdx.x == 0 && it.info && f != 0) atomicCAS((int*)it.info, 0, k0 + f);
    pivot_write(D, wave, lds, it, ws, k0, nb, k0 + NB >= d, false);
}

// The first step that tile (I, J) owes of the steps lo .. hi, and where its old values are if not where `o` says (owed_first).
__device__ __forceinline__ int owed_from(const WsView& ws, int I, int J, int lo, int hi, OldSrc& o) {
    return owed_first(I, J, lo, hi, [&](int kind, int step, int slab) { o = OldSrc{kind, ws.T(step % NBUF) + (size_t)slab * (NB * NB)}; });
}

// Tile (I, J) of a step that is not the matrix's last: brings it up to date through step g.g0 + g.j.
// single: the tile has been kept up to date step by step (a diagonal tile inside a group): it sees that step only, and its old value
// is in the working copy.  Otherwise it sees all of the group's steps up to it that it has not seen yet.
__device__ __forceinline__ void group_tile(const WsView& ws, int I, int J, const Group& g, bool single, float* __restrict__ lds) {
    const int kq = g.g0 + g.j, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
    const bool dead = I == J && wave == 1;
    OldSrc o = {OLD_W, ws.tile(I, J)};
    int first = kq;                                      // steps first .. kq, in order
    if (!single) first = owed_from(ws, I, J, g.g0, kq, o);
    TileAcc acc;
    load_old(o, dead, acc);
    if (first <= kq) {                                   // (uniform)
        const float back = tile_mma_presplit(panel_run(ws, first, kq - first + 1, I, J), (unsigned char*)lds, acc);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nbk = 0; nbk < 2; ++nbk) acc.c[mb][nbk] *= back;
    }
    if (dead) return;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nbk = 0; nbk < 2; ++nbk) store_block(tile_block(ws.tile(I, J), 2 * wm + mb, 2 * wn + nbk), acc.c[mb][nbk]);
}

// How the work list is dealt to the XCDs: equal shares, but where few matrices' look-ahead pivots run on few XCDs and the others can
// take the rest, the pivots' hosts get no more than they have compute units left (a tile's workgroup beside the pivot's lengthens
// the chain by 5 us a step).  With and without, us: one matrix of 4609 columns 1258 and 1325, two of 3073 878 and 919, three of 2305 666
// and 695, four of 2049 626 and 650; up to 325 tiles a matrix, where launches stay below a workgroup to a CU, the same within 0.5 %.
// Beyond the lines the other XCDs' second and third workgroups cost more: six matrices of 2049 columns 866 instead of 706, four of 3073
// 1292 instead of 1142, two of 4609 1661 instead of 1640 (one of 6001 columns would gain: 1768 instead of 1864).
constexpr int XCD_CUS = 32;
struct XcdShare {
    int hosts, host, other;      // XCDs 0 .. hosts - 1 get `host` workgroups each, the others `other`
};
static inline __host__ __device__ XcdShare xcd_share(int count, int total) {
    XcdShare s;
    s.hosts = 0;
    s.host = s.other = (total + 7) >> 3;
    if (count <= 4 && s.other >= XCD_CUS && s.other <= XCD_CUS * 3 / 2) {
        s.hosts = count;
        s.host = XCD_CUS - 1;
        s.other = (total - count * s.host + 7 - count) / (8 - count);
    }
    return s;
}

// One launch of the sweep: each matrix of the batch takes its stage.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(UPD_WAVES, 8))) void inv_update_kernel(ChainBatch b) {
    __shared__ __attribute__((aligned(1024))) float lds[UPD_LDS_BYTES / 4];
    __shared__ float red[4];
    // Workgroups go to the 8 XCDs round-robin (id % 8) and each XCD has an L2 of its own.  XCD x therefore takes the
    // x-th contiguous eighth of the work list (matrix by matrix: slabs, then tiles): tiles that
    // share a T panel (same block row) and mostly the same U panels run on the same L2 instead of all eight.
    // The first workgroups (one per matrix, padded to a multiple of 8 so that the others keep their XCD) take the
    // next step's pivot block; they are dispatched first and run the longest.
    const int npiv = (b.count + 7) & ~7;
    if ((int)blockIdx.x < npiv) {
        if ((int)blockIdx.x >= b.count) return;
        __builtin_amdgcn_s_setprio(3);                   // the chain's longest link: ahead of whatever shares its SIMDs
        const Item it = get_item(b, blockIdx.x);
        const int stage = b.stage[blockIdx.x];
        if (stage >= 0 && stage < nblk_of(it.dim) - 1) step_pivot(it, stage, lds);
        return;
    }
    const unsigned bx = blockIdx.x - npiv;
    const int x = bx & 7, in = bx >> 3, total = b.prefix[b.count];
    const XcdShare sh = xcd_share(b.count, total);
    const int lin = (x < sh.hosts ? x * sh.host : sh.hosts * sh.host + (x - sh.hosts) * sh.other) + in;
    if (in >= (x < sh.hosts ? sh.host : sh.other) || lin >= total) return;
    int m, tile;
    locate(b, lin, m, tile);
    const Item it = get_item(b, m);
    const int n = nblk_of(it.dim);
    const int stage = b.stage[m];
    const Plan pl = plan_of(it.dim, stage);
    if (tile < pl.slabs) {
        __builtin_amdgcn_s_setprio(2);                   // the next launch waits for these; the tiles do not hurry
        const int slab = tile >> 1, half = tile & 1;
        if (stage < n - 1) step_slab(it, stage, slab, half, lds, red);
        else last_slab(it, stage, slab, half, lds, red);
        return;
    }
    int I, J;
    bool single;
    Group g;
    if (!stage_tile(pl, n, stage, tile - pl.slabs, I, J, g, single)) return;
    group_tile(ws_view(it.ws, it.dim), I, J, g, single, lds);
}

// ---- output ----------------------------------------------------------------------------------------------------------
// One launch for all matrices of a call: every lower tile receives the last step's update (fp32 products of its nb columns), in large
// batches after the last group's (one trip through memory less; small ones, where a launch is as long as its longest workgroup, have
// these in the launch before), and its negative goes to the caller's output, with its mirror image, and, if asked for, to the piece
// planes.  (With these in launches of the sweep and the planes in a pass over the finished inverses, every tile went through memory
// twice more.)  The last group's updates here against in the launch before, us: 36 tiles (1000 columns) 284 and 273, 120 (eight
// matrices of 513) 169 and 167, 156 (two of 1500) 406 and 397, 390 (five of 1500) 450 and 441; 440 (eight of 1153) 360 and 357, 495 (nine)
// 381 and 384, 510 (34 of 513) 223 and 225, 550 (ten of 1153) 401 and 406, 561 (one of 4097) 1090 and 1104, 720 (48 of 513) 276 and 284, 1100 (twenty of
// 1153) 571 and 586; the long inversions of ResNet-50 and what runs beside them 5.23 and 5.33 ms.
// Bound: HBM.
constexpr int OMAXB = 90;
constexpr int OUT_OWED = 512;        // lower tiles of a batch from which on the output launch takes the last group's updates too
struct OutBatch {
    int count;
    int owed;                         // the last group's updates are this launch's
    int prefix[OMAXB + 1];
    int dim[OMAXB];
    float damping[OMAXB];
    const float* damping_dev[OMAXB];
    float* Minv[OMAXB];
    void* ws[OMAXB];
    void* planes[OMAXB];
};
static_assert(sizeof(OutBatch) <= 4096, "the batch travels in the kernel arguments");

struct OutPlanes {
    KFAC_AS1 unsigned char* base;    // null: none
    size_t plane;
    float scale;
};

// Elements from .. n - 1 of four neighbours, any alignment of floats.
__device__ __forceinline__ void put4(gfloat* dst, const v4f& x, int from, int n) {
    if (from <= 0 && n >= 4) {
        *(KFAC_AS1 v4f_a4*)dst = x;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i >= from && i < n) dst[i] = x[i];
    }
}

// stage (64 x SLD_T floats) holds rows h0 .. h0 + 63 of a tile's new values (zeros where the matrix ends): their negatives go out along
// the tile's rows, and along those of its mirror image.
__device__ __forceinline__ void out_flush(gfloat* __restrict__ out, const OutPlanes& pl, int d, int I, int J, int n, const float* __restrict__ stage,
                                          int h0) {
    const int t = threadIdx.x, pr = t >> 5, pc = (t & 31) * 4, i0 = I * NB, j0 = J * NB, irows = min(NB, d - i0);   // (all columns are there)
    const bool diag = I == J, planes = pl.base && !diag;
    KFAC_AS1 unsigned char* dst = pl.base + (size_t)(I * n + J) * PRE_SLAB;
    KFAC_AS1 unsigned char* mir = pl.base + (size_t)(J * n + I) * PRE_SLAB;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const int rl = pr + 8 * p, row = h0 + rl;
        v4f x;
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = -stage[rl * SLD_T + pc + i];
        if (row < irows) put4(out + (size_t)(i0 + row) * d + j0 + pc, x, 0, diag ? row - pc + 1 : 4);
        if (planes) store_split4_h2(dst, dst + pl.plane, row, pc, x * pl.scale);
    }
    const int mr = (t & 15) * 4, mc = t >> 4;             // four tile rows (neighbours in the mirror image), 16 columns a pass
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const int col = mc + 16 * p, row = h0 + mr;
        const v4f x = {-stage[mr * SLD_T + col], -stage[(mr + 1) * SLD_T + col], -stage[(mr + 2) * SLD_T + col], -stage[(mr + 3) * SLD_T + col]};
        put4(out + (size_t)(j0 + col) * d + i0 + row, x, diag ? col - row + 1 : 0, irows - row);
        if (planes) store_split4_h2(mir, mir + pl.plane, col, row, x * pl.scale);
    }
}

// The planes of diagonal block I, from the output.
__device__ __forceinline__ void out_diagonal_planes(const gfloat* __restrict__ out, const OutPlanes& pl, int d, int I, int n) {
    const int t = threadIdx.x, c4 = (t & 31) * 4, rr = t >> 5, r0 = I * NB;
    KFAC_AS1 unsigned char* dst = pl.base + (size_t)(I * n + I) * PRE_SLAB;
    v4f v[16];
    if (r0 + NB <= d) {                                   // all loads go out together (a guard per load would serialise them)
#pragma unroll
        for (int p = 0; p < 16; ++p) v[p] = *(const KFAC_AS1 v4f_a4*)(out + (size_t)(r0 + rr + 8 * p) * d + r0 + c4);
    } else {
        load_rows_edge(out, d, d, r0 + rr, r0 + c4, v);
    }
#pragma unroll
    for (int p = 0; p < 16; ++p) store_split4_h2(dst, dst + pl.plane, rr + 8 * p, c4, v[p] * pl.scale);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) void inv_out_kernel(OutBatch b) {
    __shared__ __attribute__((aligned(1024))) float lds[UPD_LDS_BYTES / 4];
    const int total = b.prefix[b.count], per_xcd = (total + 7) >> 3;             // (XCD x: the x-th contiguous eighth)
    const int lin = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || lin >= total) return;
    int m, tile, I, J;
    locate(b, lin, m, tile);
    const int d = b.dim[m], n = nblk_of(d), step = n - 1, nb = d - step * NB;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    gfloat* out = as_global(b.Minv[m]);
    OutPlanes pl;
    pl.base = (KFAC_AS1 unsigned char*)as_global((float*)b.planes[m]);
    pl.plane = inverse_plane_bytes(d);
    pl.scale = 1.f;
    tri_decode_blocked(n, tile, I, J);
    if (pl.base) {
        pl.scale = inverse_plane_scale(b.damping_dev[m] ? *as_global(b.damping_dev[m]) : b.damping[m]);
        gfloat* scales = (gfloat*)(pl.base + 2 * pl.plane);
        if (t == 0) scales[I * n + J] = scales[J * n + I] = pl.scale;
    }
    if (J == step) {                                      // the last pivot block: the pivot code wrote it
        if (pl.base) out_diagonal_planes(out, pl, d, I, n);
        return;
    }
    const WsView ws = ws_view(as_global((float*)b.ws[m]), d);
    const gfloat* T = ws.T(step % NBUF);
    if (I == step) {                                      // block row of the last step: T, transposed
#pragma unroll 1
        for (int h0 = 0; h0 < NB; h0 += 64) {             // (rows beyond nb: zeros, for the planes)
            if (h0 > 0) __syncthreads();
            const int ta = (t & 15) * 4, tc = t >> 4;     // 16 float4 along the tile's rows, 16 columns a pass
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int cc = tc + 16 * p;
                const v4f x = *(const KFAC_AS1 v4f*)&T[(size_t)(J * NB + cc) * NB + h0 + ta];
#pragma unroll
                for (int i = 0; i < 4; ++i) lds[(ta + i) * SLD_T + cc] = h0 + ta + i < nb ? x[i] : 0.f;
            }
            __syncthreads();
            out_flush(out, pl, d, I, J, n, lds, h0);
        }
        return;
    }
    // The last group's steps, as in group_tile, then the last step.
    const int h = lane >> 5;
    const bool dead = I == J && wave == 1;
    OldSrc o = {OLD_W, ws.tile(I, J)};
    const int first = b.owed ? owed_from(ws, I, J, (step - 1) / GM * GM, step - 1, o) : step;
    TileAcc acc, last;
    load_old(o, dead, acc);
    if (first < step) {                                   // (uniform)
        const float back = tile_mma_presplit(panel_run(ws, first, step - first, I, J), (unsigned char*)lds, acc);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nbk = 0; nbk < 2; ++nbk) acc.c[mb][nbk] *= back;
    }
    product_f32(T + (size_t)I * (NB * NB), ws.U(step % NBUF) + (size_t)J * (NB * NB), nb, dead, lds, last);
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        if (half == 1) __syncthreads();
        if (wm == half) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nbk = 0; nbk < 2; ++nbk)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        lds[(mb * 32 + (r >> 2) * 8 + h * 4 + (r & 3)) * SLD_T + acc_col(wn, nbk, lane)] = acc.c[mb][nbk][r] - last.c[mb][nbk][r];
        }
        __syncthreads();
        out_flush(out, pl, d, I, J, n, lds, half * 64);
    }
    if (I == J && pl.base) {
        __threadfence_block();
        __syncthreads();                                  // the block is in the output, both triangles
        out_diagonal_planes(out, pl, d, I, n);
    }
}

static int write_outputs(const kfac_inverse_item* h, int count, bool owed, hipStream_t stream) {
    OutBatch b;
    b.owed = owed;
    for (int first = 0; first < count; first += OMAXB) {
        b.count = min(OMAXB, count - first);
        b.prefix[0] = 0;
        for (int i = 0; i < b.count; ++i) {
            const kfac_inverse_item& it = h[first + i];
            const int n = nblk_of(it.dim);
            b.dim[i] = it.dim; b.damping[i] = it.damping; b.damping_dev[i] = it.damping_dev;
            b.Minv[i] = it.Minv; b.ws[i] = it.ws; b.planes[i] = it.planes;
            b.prefix[i + 1] = b.prefix[i] + (n > 1 || it.planes ? n * (n + 1) / 2 : 0);
        }
        if (b.prefix[b.count] > 0) KFAC_LAUNCH(inv_out_kernel, dim3(8 * ((b.prefix[b.count] + 7) / 8)), dim3(256), stream, b);
    }
    return KFAC_OK;
}

static void fill_batch(Batch& b, const kfac_inverse_item* items, int count) {
    b.count = count;
    for (int i = 0; i < count; ++i) {
        b.dim[i] = items[i].dim;
        b.damping[i] = items[i].damping;
        b.damping_dev[i] = items[i].damping_dev;
        b.S[i] = items[i].S;
        b.Minv[i] = items[i].Minv;
        b.ws[i] = items[i].ws;
        b.info[i] = items[i].info;
    }
}

// items must be sorted by non-increasing dim (checked by the caller of this function).
static int run_group(const kfac_inverse_item* h, int count, hipStream_t stream) {
    Batch b;
    // matrices needing the blocked path (more than one block) come first in the sorted order
    int n_multi = 0;
    while (n_multi < count && nblk_of(h[n_multi].dim) > 1) ++n_multi;

    for (int first = 0; first < count; first += MAXB) {
        const int n = min(MAXB, count - first);
        fill_batch(b, h + first, n);
        b.prefix[0] = 0;
        for (int i = 0; i < n; ++i) b.prefix[i + 1] = b.prefix[i] + begin_workgroups(nblk_of(h[first + i].dim));
        const bool together = b.prefix[n] <= BEGIN_TOGETHER;
        if (!together) KFAC_LAUNCH(inv_init_kernel, dim3(b.prefix[n]), dim3(256), stream, b);
        KFAC_LAUNCH(inv_begin_kernel, dim3(n + (together ? b.prefix[n] : 0)), dim3(256), stream, b);
    }
    if (n_multi == 0) return write_outputs(h, count, false, stream);
    int tiles = 0;
    for (int i = 0; i < n_multi; ++i) tiles += nblk_of(h[i].dim) * (nblk_of(h[i].dim) + 1) / 2;
    const bool out_owed = tiles >= OUT_OWED;
    // One launch per stage of the matrix with the most blocks.  A matrix with fewer blocks takes
    // its stages at evenly spread launches rather than in the first ones: the tile updates of the whole batch are then
    // spread over all launches, each of which lasts at least as long as a pivot workgroup anyway.
    ChainBatch c;
    c.count = n_multi;
    c.prefix[0] = 0;
    for (int i = 0; i < n_multi; ++i) {
        c.dim[i] = h[i].dim; c.Minv[i] = h[i].Minv; c.ws[i] = h[i].ws; c.info[i] = h[i].info;
    }
    int done[CMAXB] = {};                               // stages taken so far
    const int launches = nblk_of(h[0].dim);
    for (int l = 0; l < launches; ++l) {
        for (int i = 0; i < n_multi; ++i) {
            const bool run = takes_stage(nblk_of(h[i].dim), launches, i, l);
            c.stage[i] = run ? done[i] : -1;
            c.prefix[i + 1] = c.prefix[i] + (run ? plan_workgroups(plan_of(h[i].dim, done[i]), out_owed) : 0);
            done[i] += run;
        }
        const XcdShare sh = xcd_share(n_multi, c.prefix[n_multi]);
        KFAC_LAUNCH(inv_update_kernel, dim3(((n_multi + 7) & ~7) + 8 * max(sh.host, sh.other)), dim3(256), stream, c);
    }
    return write_outputs(h, count, out_owed, stream);
}

static size_t ws_bytes_of(int dim) {
    if (nblk_of(dim) == 1) return 256;
    return align_up((working_copy_floats(dim) + NBUF * panel_buffer_floats(dim) + (size_t)2 * NB * NB + 4 * NBUF * (size_t)nblk_of(dim)) * sizeof(float), 256);
}

static bool item_ok(const kfac_inverse_item& it) {
    if (!it.S || !it.Minv || it.dim <= 0 || it.dim > 32768) return false;
    if (it.S == it.Minv) return false;
    if (nblk_of(it.dim) > 1 && (!it.ws || ((uintptr_t)it.ws & 255))) return false;
    if (it.planes && (((uintptr_t)it.planes & 255) || (!it.damping_dev && !(it.damping > 0.f)))) return false;
    return true;
}

}  // namespace kfac

using namespace kfac;

extern "C" size_t kfac_inverse_workspace_bytes(int32_t dim) {
    if (dim <= 0 || dim > 32768) return 0;
    return ws_bytes_of(dim);
}

extern "C" size_t kfac_inverse_planes_bytes(int32_t dim) {
    if (dim <= 0 || dim > 32768) return 0;
    return align_up(inverse_planes_bytes(dim), 256);
}

extern "C" int kfac_damped_inverse(const float* S, int32_t dim, float damping, float* Minv, int32_t* info,
                                   void* ws, size_t ws_bytes, void* stream) {
    kfac_inverse_item it;
    it.S = S; it.Minv = Minv; it.ws = ws; it.info = info; it.dim = dim; it.damping = damping; it.damping_dev = nullptr;
    it.planes = nullptr;
    if (dim <= 0 || dim > 32768 || !S || !Minv || S == Minv) return KFAC_ERR_INVALID_ARG;
    if (nblk_of(dim) > 1) {
        if (!ws || ((uintptr_t)ws & 255) || ws_bytes < ws_bytes_of(dim)) return KFAC_ERR_WORKSPACE;
    }
    return run_group(&it, 1, (hipStream_t)stream);
}

extern "C" int kfac_damped_inverse_batched(const kfac_inverse_item* items_host, int32_t count, void* stream) {
    if (count == 0) return KFAC_OK;                       // nothing to do, no launch
    if (!items_host || count < 0) return KFAC_ERR_INVALID_ARG;
    for (int i = 0; i < count; ++i) {
        if (!item_ok(items_host[i])) return KFAC_ERR_INVALID_ARG;
        if (i > 0 && items_host[i].dim > items_host[i - 1].dim) return KFAC_ERR_INVALID_ARG;   // sorted, largest first
    }
    // Matrices beyond what one launch's argument block can describe go into further groups.  Dealing them round
    // robin keeps every group's size mix (and hence its step count and load) similar.
    const int ngroups = (count + CMAXB - 1) / CMAXB;
    for (int g = 0; g < ngroups; ++g) {
        kfac_inverse_item sel[CMAXB];
        int n = 0;
        for (int i = g; i < count; i += ngroups) sel[n++] = items_host[i];
        int rc = run_group(sel, n, (hipStream_t)stream);
        if (rc != KFAC_OK) return rc;
    }
    return KFAC_OK;
}
