// fp32 products on the 16-bit matrix cores, operands split into 16-bit pieces.
//
// Three bf16 pieces (the sweep's panel product, below): each fp32 operand value is split on the fly,
//     x = x0 + x1 + x2,   x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1)
// (8 significant bits each, all 24 of x together), and the product is the sum of the bf16 x bf16 MFMAs (exact products, fp32
// accumulate) of all piece pairs whose combined order is below 3:
//     a0 b0 + a0 b1 + a1 b0 + a0 b2 + a1 b1 + a2 b0     relative error ~ 2^-23: on a par with fp32 multiply-add
// v_mfma_f32_32x32x16_bf16 runs at 16 times the rate of v_mfma_f32_32x32x2_f32, so 6 products per fp32 product still leave a
// factor 2.7 over the fp32 matrix-core peak.
//
// Two fp16 pieces of scaled operands, split ahead of time by their producer: the rest of the file.
#pragma once

#include "factor_mfma.h"
#include "gemm_f32.h"

namespace kfac {

constexpr int SPLIT_KS = 16;                           // K per LDS stage
constexpr int SPLIT_PLANE = 128 * 32;                  // bytes of one operand piece per stage

typedef __bf16 v2bf_t __attribute__((ext_vector_type(2)));
typedef float v2f_t __attribute__((ext_vector_type(2)));

// bf16 pieces of four floats: piece[p] holds 4 bf16 (8 bytes) for p < NS
template <int NS>
__device__ __forceinline__ void split4(const v4f& x, uint2 (&piece)[NS]) {
    v4f rem = x;
#pragma unroll
    for (int p = 0; p < NS; ++p) {
        const v2f_t lo2 = {rem.x, rem.y}, hi2 = {rem.z, rem.w};
        const v2bf_t a = __builtin_convertvector(lo2, v2bf_t), b = __builtin_convertvector(hi2, v2bf_t);
        unsigned ua, ub;
        __builtin_memcpy(&ua, &a, 4);
        __builtin_memcpy(&ub, &b, 4);
        piece[p] = make_uint2(ua, ub);
        if (p + 1 < NS) {
            rem.x -= __uint_as_float(ua << 16);
            rem.y -= __uint_as_float(ua & 0xffff0000u);
            rem.z -= __uint_as_float(ub << 16);
            rem.w -= __uint_as_float(ub & 0xffff0000u);
        }
    }
}

// acc[64 x 128] = A[64 x 128] . B[128 x 128]^T for a workgroup of 4 wavefronts, each owning 32 rows x 64 columns as two
// MFMA blocks.  A: complete rows in global memory, leading dimension 128.  B passes through LDS: its values are fetched by
// panel_fetch_b (any time before: the caller hides the latency), split a 16-wide slice at a time and stored to a
// double-buffered stage of 3 pieces x 128 rows x 32 bytes; the two 16-byte halves of a row swap places from one group of 4
// rows to the next and again from one group of 8 to the next, which makes the 16-byte MFMA operand reads (served 16
// consecutive rows at a time from 64 banks) bank-conflict free.  A's 8 values per lane and slice are the lane's operand as they
// lie in memory: split in registers, two slices ahead in flight.  lds: PANEL_B_LDS bytes, 16-byte aligned; one barrier a slice.
constexpr int PANEL_B_LDS = 2 * 3 * SPLIT_PLANE;

// B's rows lr and lr + 64 (lr = t / 4), floats 4 kq .. + 3 (kq = t % 4) of slice s: fetched, and stored as pieces to stage s % 2.
__device__ __forceinline__ void panel_fetch_slice(const gfloat* __restrict__ B, int s, v4f (&x)[2]) {
    const int lr = threadIdx.x >> 2, kq = threadIdx.x & 3;
#pragma unroll
    for (int p = 0; p < 2; ++p) x[p] = *(const KFAC_AS1 v4f*)(B + (lr + 64 * p) * 128 + s * SPLIT_KS + 4 * kq);
}

__device__ __forceinline__ void panel_stash(unsigned char* __restrict__ lds, int s, const v4f (&x)[2]) {
    const int lr = threadIdx.x >> 2, kq = threadIdx.x & 3;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int row = lr + 64 * p;
        const unsigned off = (unsigned)(row * 32 + (((kq >> 1) ^ ((row >> 2) & 1) ^ ((row >> 3) & 1)) * 16) + (kq & 1) * 8);
        uint2 piece[3];
        split4<3>(x[p], piece);
#pragma unroll
        for (int e = 0; e < 3; ++e) *(uint2*)(lds + (s & 1) * (3 * SPLIT_PLANE) + e * SPLIT_PLANE + off) = piece[e];
    }
}

__device__ __forceinline__ void panel_fetch_b(const gfloat* __restrict__ B, v4f (&pb)[8][2]) {
#pragma unroll
    for (int s = 0; s < 8; ++s) panel_fetch_slice(B, s, pb[s]);
}

__device__ __forceinline__ void panel_product(const gfloat* __restrict__ A, const v4f (&pb)[8][2], unsigned char* __restrict__ lds,
                                              v16f (&acc)[2]) {
    constexpr int BUF = 3 * SPLIT_PLANE;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const int lm = lane & 31, h = lane >> 5;
    unsigned b_off[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int rb = wn * 64 + p * 32 + lm;
        b_off[p] = (unsigned)(rb * 32 + ((h ^ ((rb >> 2) & 1) ^ ((rb >> 3) & 1)) * 16));
    }
    v4f xa[3][2];                                                // slices s, s + 1, s + 2
    const gfloat* arow = A + (wm * 32 + lm) * 128 + 8 * h;
    auto fetch = [&](int s, v4f (&x)[2]) {
        x[0] = *(const KFAC_AS1 v4f*)(arow + s * SPLIT_KS);
        x[1] = *(const KFAC_AS1 v4f*)(arow + s * SPLIT_KS + 4);
    };
    fetch(0, xa[0]);
    fetch(1, xa[1]);
    panel_stash(lds, 0, pb[0]);
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[n][r] = 0.f;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        if (s + 2 < 8) fetch(s + 2, xa[(s + 2) % 3]);
        uint4 a[3], b[2][3];
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int e = 0; e < 3; ++e) b[n][e] = *(const uint4*)(lds + (s & 1) * BUF + e * SPLIT_PLANE + b_off[n]);
        uint2 lo[3], hi[3];
        split4<3>(xa[s % 3][0], lo);
        split4<3>(xa[s % 3][1], hi);
#pragma unroll
        for (int e = 0; e < 3; ++e) a[e] = make_uint4(lo[e].x, lo[e].y, hi[e].x, hi[e].y);
        // smallest terms first
#pragma unroll
        for (int order = 2; order >= 0; --order)
#pragma unroll
            for (int pa = 0; pa <= order; ++pa)
#pragma unroll
                for (int n = 0; n < 2; ++n) acc[n] = mfma16<false>(a[pa], b[n][order - pa], acc[n]);
        if (s + 1 < 8) panel_stash(lds, s + 1, pb[s + 1]);
        __syncthreads();
    }
}

// ---- two fp16 pieces ---------------------------------------------------------------------------------------------
// x = h0 + h1 with h0 = fp16(x), h1 = fp16(x - h0): 11 significant bits each, 22 together, and the three piece
// products h0 h0 + h0 h1 + h1 h0 (exact in the fp32 accumulator) leave a relative error of ~2^-22 per product: on a
// par with fp32 for a sum of 128 terms, at half the matrix-core work and two thirds of the LDS traffic of three bf16
// pieces.  fp16 has a narrow exponent range, so every operand panel comes with a power-of-two scale that brings its
// largest magnitude to about 2^8 (smaller entries then lose bits only below 2^-32 of the largest); the caller scales the accumulators to match (exact) and back afterwards.
typedef _Float16 v2h_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void split4_h2(const v4f& x, uint2 (&piece)[2]) {
    v4f rem = x;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const v2f_t lo2 = {rem.x, rem.y}, hi2 = {rem.z, rem.w};
        const v2h_t a = __builtin_convertvector(lo2, v2h_t), b = __builtin_convertvector(hi2, v2h_t);
        unsigned ua, ub;
        __builtin_memcpy(&ua, &a, 4);
        __builtin_memcpy(&ub, &b, 4);
        piece[p] = make_uint2(ua, ub);
        if (p == 0) {
            const v2f_t la = __builtin_convertvector(a, v2f_t), lb = __builtin_convertvector(b, v2f_t);
            rem.x -= la.x; rem.y -= la.y; rem.z -= lb.x; rem.w -= lb.y;
        }
    }
}

// Scale (a power of two, as a float) that brings a panel whose largest magnitude is `amax` to at most 2^8: fp16 has
// seven binades above that before it overflows, and the further up the values sit, the later their low pieces
// (2^-11 of the value) drop into fp16's subnormal range: entries down to 2^-11 of the largest keep all 22 bits.
// Exponents are kept within +-30 so that products of two scales and their reciprocals stay far from the ends of the
// fp32 range.
constexpr int PANEL_TOP = 8;
__device__ __forceinline__ float panel_scale(float amax) {
    int e = 0;
    if (amax > 0.f) {
        (void)frexpf(amax, &e);                        // amax = m 2^e, 0.5 <= m < 1
        e = max(-30, min(30, e));
    }
    return ldexpf(1.0f, PANEL_TOP - e);
}

// Largest of the 256 threads' values (red: 4 floats of LDS); two barriers.  Must be called by all threads.
__device__ __forceinline__ float block_absmax(float x, float* __restrict__ red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    x = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    return x;
}

// ---- operands split ahead of time ----------------------------------------------------------------------------------
// A panel (128-row slabs x 128 columns of the contraction index) that many tile products read is scaled and split
// into its two fp16 pieces once, by the kernel that produces it, instead of by every product that consumes it: the
// consumer then has no conversion work at all and moves the pieces from global memory straight into LDS
// (global_load_lds_dwordx4: lane i's 16 bytes land at base + 16 i, no registers involved).  To make those copies
// whole contiguous kilobytes, a piece plane is stored in the order the product wants it in LDS: slab by slab, and
// inside a slab one 4 KB block per 16-wide slice of the contraction index, holding for every row its two 16-byte
// halves (8 fp16 each) at byte offset split_plane_offset(row, half).  The halves swap places from one group of four rows
// to the next and again from one group of eight to the next: a 16-byte operand read is served 16 lanes (consecutive rows)
// at a time from 64 four-byte banks, and with this order any 16 consecutive rows' halves fall into 16 different
// 16-byte bank groups (so do any 8 rows' in 8 of 32 banks); with rows simply 32 bytes apart, rows r and r + 8 collide.
constexpr int PRE_BLOCK = 128 * SPLIT_KS * 2;          // bytes of one (slab, 16-wide slice) block of one piece plane
constexpr int PRE_SLAB = (128 / SPLIT_KS) * PRE_BLOCK; // bytes of one 128 x 128 slab of one piece plane
constexpr int PRE_STAGE = 4 * PRE_BLOCK;               // LDS per ring stage: A high, A low, B high, B low
constexpr int PRE_NS = 3;                              // ring stages (two in flight)

__host__ __device__ __forceinline__ int split_plane_offset(int row, int half) {
    return row * 32 + ((half ^ ((row >> 2) & 1) ^ ((row >> 3) & 1)) * 16);
}

// Scaled fp16 pieces of four consecutive contraction-index values k4 .. k4 + 3 (k4 a multiple of 4) of one row of a
// slab, written to the planes `hi` / `lo` (pointing at the slab).
__device__ __forceinline__ void store_split4_h2(KFAC_AS1 unsigned char* hi, KFAC_AS1 unsigned char* lo, int row, int k4,
                                                const v4f& x_scaled) {
    uint2 piece[2];
    split4_h2(x_scaled, piece);
    const int off = (k4 >> 4) * PRE_BLOCK + split_plane_offset(row, (k4 >> 3) & 1) + (k4 & 7) * 2;
    typedef unsigned v2u_t __attribute__((ext_vector_type(2)));
    *(KFAC_AS1 v2u_t*)(hi + off) = v2u_t{piece[0].x, piece[0].y};
    *(KFAC_AS1 v2u_t*)(lo + off) = v2u_t{piece[1].x, piece[1].y};
}

// The rank-128 products of a tile.  The operands of consecutive products sit in consecutive buffers of a ring of `nbuf`
// equally laid out buffers `stride` bytes apart: product q reads buffer (first + q) mod nbuf, the
// high pieces of its A slab at a_hi + buffer * stride, the low pieces `plane` bytes further, and likewise b_hi;
// scale[q] = sa * sb is what the product of the stored pieces is scaled by.
template <int MAXN>
struct SplitRun {
    const KFAC_AS1 unsigned char* a_hi;                // in buffer 0
    const KFAC_AS1 unsigned char* b_hi;
    size_t plane;                                      // bytes from a high plane to its low plane
    size_t stride;                                     // bytes from one buffer to the next
    float scale[MAXN];
    int first, nbuf;
    int n;                                             // 1 .. MAXN products
};

// Brings accumulators from scale 1 / back to scale sq (powers of two, the same in all lanes of the wavefront); back becomes 1 / sq.
// Neighbouring products often have the same scale: then there is nothing to do.
template <class Acc>
__device__ __forceinline__ void rescale(float sq, float& back, Acc&& multiply_all) {
    sq = uniform(sq);
    const float f = sq * back;
    if (f != 1.0f) multiply_all(f);
    back = __uint_as_float(0x7F000000u - __float_as_uint(sq));     // (of a power of two between 2^-126 and 2^126)
}

// The loop of the tile products: acc[128 x 128] (+)= sum over nst 16-wide slices.  issue(s, buf): this wavefront's four copies of
// slice s into ring stage buf; begin(s): called before a product's first slice is multiplied.
// A slice's operands are read from LDS while the slice before is multiplied, so the ring's three stages hold one slice that is being
// read and two that are on their way (110 tile products a microsecond on the chip, 98 with each slice read before it is multiplied; four
// to a visit of a tile in W included 86 against 83).  All 256 threads must call; ends with the ring drained and a barrier.
template <class Issue, class Begin>
__device__ __forceinline__ void tile_mma_loop(int nst, Issue&& issue, Begin&& begin, TileAcc& acc) {
    constexpr int NSL = 128 / SPLIT_KS;                // slices per product
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1;
    const int lm = lane & 31, h = lane >> 5;
    unsigned a_addr[2], b_addr[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        a_addr[q] = (unsigned)split_plane_offset(wm * 64 + q * 32 + lm, h);
        b_addr[q] = (unsigned)(2 * PRE_BLOCK + split_plane_offset(wn * 64 + q * 32 + lm, h));
    }
    v4f a[2][2][2], b[2][2][2];                        // [set][block][piece] (16 bytes = 8 fp16 each)
    auto read = [&](int set, int stage) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int pc = 0; pc < 2; ++pc) {
                // (the stage's base goes into the address: an instruction offset holds 16 bits only)
                asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(a[set][q][pc]) : "v"(a_addr[q] + stage * PRE_STAGE), "n"(pc * PRE_BLOCK));
                asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(b[set][q][pc]) : "v"(b_addr[q] + stage * PRE_STAGE), "n"(pc * PRE_BLOCK));
            }
    };
    static_assert(PRE_NS == 3, "the waits below count younger copies");
#pragma unroll
    for (int s = 0; s < PRE_NS; ++s) issue(s, s);
    asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
    read(0, 0);
    for (int it = 0; it < nst; it += 2 * PRE_NS) {
#pragma unroll
        for (int bi = 0; bi < 2 * PRE_NS; ++bi) {
            const int s = it + bi;
            if (s >= nst) break;                                            // uniform
            // slice s is in registers, slice s + 1 landed (everybody's part): the place of slice s is free
            const int set = bi & 1;
            asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier"
                         : "+v"(a[set][0][0]), "+v"(a[set][0][1]), "+v"(a[set][1][0]), "+v"(a[set][1][1]),
                           "+v"(b[set][0][0]), "+v"(b[set][0][1]), "+v"(b[set][1][0]), "+v"(b[set][1][1]) :: "memory");
            read(set ^ 1, (bi + 1) % PRE_NS);
            issue(s + PRE_NS, bi % PRE_NS);
            if (s % NSL == 0) begin(s);
            // smallest terms first
#pragma unroll
            for (int term = 0; term < 3; ++term)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) {
                        v8h av, bv;
                        __builtin_memcpy(&av, &a[set][mb][term == 0 ? 1 : 0], 16);
                        __builtin_memcpy(&bv, &b[set][nb][term == 1 ? 1 : 0], 16);
                        acc.c[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv, acc.c[mb][nb], 0, 0, 0);
                    }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // (the last read's registers are not free before that wait)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier"
                 : "+v"(a[0][0][0]), "+v"(a[0][0][1]), "+v"(a[0][1][0]), "+v"(a[0][1][1]),
                   "+v"(b[0][0][0]), "+v"(b[0][0][1]), "+v"(b[0][1][0]), "+v"(b[0][1][1]) :: "memory");
}

// acc[128 x 128] (+)= sum over the products q of A_q B_q^T, A_q / B_q complete 128 x 128 slabs given as piece planes
// (high x high + high x low + low x high on the fp16 matrix cores).  The products may be scaled differently: acc is
// brought to product q's scale before it is added to (acc holds the caller's values, at scale 1, on entry), and the
// returned factor brings it back to scale 1 (the caller multiplies).  lds: PRE_NS * PRE_STAGE bytes, 1 KB aligned.
template <int MAXN>
__device__ __forceinline__ float tile_mma_presplit(const SplitRun<MAXN>& p, unsigned char* __restrict__ lds, TileAcc& acc) {
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    constexpr int NSL = 128 / SPLIT_KS;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_byte* l0 = (lds_byte*)lds;
    const int nst = p.n * NSL;
    const unsigned lane_off = (unsigned)(wave * 1024 + lane * 16);   // this lane's 16 bytes inside every block
    float back = 1.0f;
    tile_mma_loop(nst, [&](int s, int buf) {
        const int sc = s < nst ? s : nst - 1;          // past the end: re-read the last slice (never consumed)
        const int q = sc / NSL, ks = sc - q * NSL;
        const int bq = p.first + q;                    // (first < nbuf, q < nbuf)
        const size_t boff = (size_t)(bq >= p.nbuf ? bq - p.nbuf : bq) * p.stride;
        const KFAC_AS1 unsigned char* pa = p.a_hi + boff;
        const KFAC_AS1 unsigned char* pb = p.b_hi + boff;
        const KFAC_AS1 unsigned char* src[4] = {pa, pa + p.plane, pb, pb + p.plane};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + ks * PRE_BLOCK + lane_off),
                                             (__attribute__((address_space(3))) void*)(l0 + buf * PRE_STAGE + j * PRE_BLOCK + wave * 1024),
                                             16, 0, 0);
    }, [&](int s) {
        float sq = p.scale[0];
#pragma unroll
        for (int q = 1; q < MAXN; ++q) sq = s / NSL == q ? p.scale[q] : sq;
        rescale(sq, back, [&](float f) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) acc.c[mb][nb] *= f;
        });
    }, acc);
    return back;
}

// The same for half a slab of A: acc[64 x 128] (+)= sum over the products of A_q B_q^T, A's planes pointing at the half slab's rows.
// Wavefront (wm, wn) holds rows 32 wm .. + 31 of columns 64 wn .. + 63 as two MFMA blocks.  A slice is 12 KB, three 1 KB copies a
// wavefront (kilobytes 3 wave .. + 2 of a stage: 0, 1 A high, 2, 3 A low, 4 .. 7 B high, 8 .. 11 B low), in a ring of HALF_NS stages: one
// being read, three on their way.
constexpr int HALF_STAGE = 3 * PRE_BLOCK;              // A high, A low (half a block each), B high, B low
constexpr int HALF_NS = 4;

struct HalfCopies {
    const KFAC_AS1 unsigned char* src[3];              // in slice 0 of product 0
};
__device__ __forceinline__ HalfCopies half_copies(const KFAC_AS1 unsigned char* a_hi, size_t a_plane, const KFAC_AS1 unsigned char* b_hi,
                                                  size_t b_plane) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    HalfCopies c;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int kb = 3 * wave + j;
        c.src[j] = (kb < 4 ? a_hi + (kb >> 1) * a_plane + (kb & 1) * 1024 : b_hi + (kb >= 8 ? b_plane : 0) + (kb & 3) * 1024) + lane * 16;
    }
    return c;
}
// The three copies of the slice that lies `off` bytes further in both operands' planes.
__device__ __forceinline__ void half_issue(const HalfCopies& c, size_t off, unsigned char* __restrict__ lds, int buf) {
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int j = 0; j < 3; ++j)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(c.src[j] + off),
                                         (__attribute__((address_space(3))) void*)((lds_byte*)lds + buf * HALF_STAGE + (3 * wave + j) * 1024),
                                         16, 0, 0);
}

template <class Issue, class Begin>
__device__ __forceinline__ void half_mma_loop(int nst, Issue&& issue, Begin&& begin, v16f (&acc)[2]) {
    constexpr int NSL = 128 / SPLIT_KS;
    static_assert(HALF_NS == 4 && NSL % HALF_NS == 0, "the waits below count younger copies; nst is a multiple of HALF_NS");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 1, wn = wave & 1, lm = lane & 31, h = lane >> 5;
    const unsigned a_addr = (unsigned)split_plane_offset(wm * 32 + lm, h);
    unsigned b_addr[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) b_addr[q] = (unsigned)(PRE_BLOCK + split_plane_offset(wn * 64 + q * 32 + lm, h));
    v4f a[2][2], b[2][2][2];                           // [set][piece], [set][block][piece] (16 bytes = 8 fp16 each)
    auto read = [&](int set, int stage) {
        asm volatile("ds_read_b128 %0, %1" : "=v"(a[set][0]) : "v"(a_addr + stage * HALF_STAGE));
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(a[set][1]) : "v"(a_addr + stage * HALF_STAGE), "n"(PRE_BLOCK / 2));
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int pc = 0; pc < 2; ++pc)
                asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(b[set][q][pc]) : "v"(b_addr[q] + stage * HALF_STAGE), "n"(pc * PRE_BLOCK));
    };
#pragma unroll
    for (int s = 0; s < HALF_NS; ++s) issue(s, s);
    asm volatile("s_waitcnt vmcnt(9)\n\ts_barrier" ::: "memory");
    read(0, 0);
    for (int it = 0; it < nst; it += HALF_NS) {
#pragma unroll
        for (int bi = 0; bi < HALF_NS; ++bi) {
            const int s = it + bi, set = bi & 1;
            // slice s is in registers, slice s + 1 landed (everybody's part): the place of slice s is free
            asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier"
                         : "+v"(a[set][0]), "+v"(a[set][1]), "+v"(b[set][0][0]), "+v"(b[set][0][1]), "+v"(b[set][1][0]), "+v"(b[set][1][1]) :: "memory");
            read(set ^ 1, (bi + 1) % HALF_NS);
            issue(s + HALF_NS, bi);
            if (s % NSL == 0) begin(s);                                      // (uniform: a new product)
            // smallest terms first
#pragma unroll
            for (int term = 0; term < 3; ++term)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    v8h av, bv;
                    __builtin_memcpy(&av, &a[set][term == 0 ? 1 : 0], 16);
                    __builtin_memcpy(&bv, &b[set][nb][term == 1 ? 1 : 0], 16);
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv, acc[nb], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // (the last read's registers are not free before that wait)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier"
                 : "+v"(a[0][0]), "+v"(a[0][1]), "+v"(b[0][0][0]), "+v"(b[0][0][1]), "+v"(b[0][1][0]), "+v"(b[0][1][1]) :: "memory");
}

constexpr int HALF_MAXN = 5;
typedef SplitRun<HALF_MAXN> HalfRun;                   // (scale[q]: that of the wavefront's columns)

__device__ __forceinline__ float half_mma_presplit(const HalfRun& p, unsigned char* __restrict__ lds, v16f (&acc)[2]) {
    constexpr int NSL = 128 / SPLIT_KS;
    const HalfCopies c = half_copies(p.a_hi, p.plane, p.b_hi, p.plane);
    const int nst = p.n * NSL;
    float back = 1.0f;
    half_mma_loop(nst, [&](int s, int buf) {
        const int sc = s < nst ? s : nst - 1;          // past the end: re-read the last slice (never consumed)
        const int q = sc / NSL, ks = sc - q * NSL;
        const int bq = p.first + q;                    // (first < nbuf, q < nbuf)
        const size_t off = (size_t)(bq >= p.nbuf ? bq - p.nbuf : bq) * p.stride + ks * PRE_BLOCK;
        half_issue(c, off, lds, buf);
    }, [&](int s) {
        float sq = p.scale[0];
#pragma unroll
        for (int q = 1; q < HALF_MAXN; ++q) sq = s / NSL == q ? p.scale[q] : sq;
        rescale(sq, back, [&](float f) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc[nb] *= f;
        });
    }, acc);
    return back;
}

// A long contraction: product q reads the q-th consecutive 128 x 128 block of its operands' planes (the blocks of one
// 128-row slab of a matrix stored block by block along the contraction index); scale_lds[q] (LDS, filled and made
// visible by the caller) is the product of the two blocks' scales, for the wavefront's columns.
struct SplitSeq {
    const KFAC_AS1 unsigned char* a_hi;                // first block of the A slab's high plane
    const KFAC_AS1 unsigned char* b_hi;
    size_t plane_a, plane_b;                           // bytes from each operand's high plane to its low plane
    const float* scale_lds;
    int n;
    __device__ __forceinline__ float scale_of(int q) const { return scale_lds[q]; }
};

// The same for a long contraction given as a SplitSeq.  (With its addresses in scalar registers the preconditioner has room for the
// second set of operands; before, 16 registers went to scratch memory and a slice was read just before it was multiplied: both products of ResNet-50 592 -> 544 us.)
__device__ __forceinline__ float tile_mma_presplit_seq(const SplitSeq& p, unsigned char* __restrict__ lds, TileAcc& acc) {
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    constexpr int NSL = 128 / SPLIT_KS;                // slices per product
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds_byte* l0 = (lds_byte*)lds;
    const int nst = p.n * NSL;
    const unsigned lane_off = (unsigned)(wave * 1024 + lane * 16);   // this lane's 16 bytes inside every block
    float back = 1.0f;
    tile_mma_loop(nst, [&](int s, int buf) {
        const int sc = s < nst ? s : nst - 1;          // past the end: re-read the last slice (never consumed)
        const size_t off = (size_t)(sc / NSL) * PRE_SLAB + (sc % NSL) * PRE_BLOCK;
        const KFAC_AS1 unsigned char* src[4] = {p.a_hi + off, p.a_hi + p.plane_a + off, p.b_hi + off, p.b_hi + p.plane_b + off};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + lane_off),
                                             (__attribute__((address_space(3))) void*)(l0 + buf * PRE_STAGE + j * PRE_BLOCK + wave * 1024),
                                             16, 0, 0);
    }, [&](int s) {
        rescale(p.scale_of(s / NSL), back, [&](float f) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) acc.c[mb][nb] *= f;
        });
    }, acc);
    return back;
}

// The same for half a slab of A (a_hi pointing at the half slab's rows).
__device__ __forceinline__ float half_mma_presplit_seq(const SplitSeq& p, unsigned char* __restrict__ lds, v16f (&acc)[2]) {
    constexpr int NSL = 128 / SPLIT_KS;
    const HalfCopies c = half_copies(p.a_hi, p.plane_a, p.b_hi, p.plane_b);
    const int nst = p.n * NSL;
    float back = 1.0f;
    half_mma_loop(nst, [&](int s, int buf) {
        const int sc = s < nst ? s : nst - 1;          // past the end: re-read the last slice (never consumed)
        const int q = sc / NSL, ks = sc - q * NSL;
        const size_t off = (size_t)q * PRE_SLAB + ks * PRE_BLOCK;
        half_issue(c, off, lds, buf);
    }, [&](int s) {
        const float sq = p.scale_of(s / NSL);
        rescale(sq, back, [&](float f) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc[nb] *= f;
        });
    }, acc);
    return back;
}

}  // namespace kfac
