// Matrix-core factor builder: tiles of  Xbar^T Xbar  straight from a channels-last tensor (or NCHW planes: FEED_PLANES), Xbar the
// implicitly unfolded patch matrix, for 16-bit inputs and, in three bf16 pieces, fp32 ones (v_mfma_f32_32x32x16 both).
//
// One TW x TW tile (on or below the diagonal) of one range of unfolded rows per workgroup.  The contraction index (the
// unfolded row) is the slow index in memory, and the 16-bit MFMA wants it contiguous per lane; gfx950 has exactly the two
// instructions that make this cheap:
//   * a load to LDS copies 16 bytes per lane from global memory (lane i lands at base + 16 i) without passing through registers, so a ring
//     of row slabs can be kept in flight with no register cost and a single barrier per slab: buffer_load_dwordx4 .. lds from 32-bit offsets
//     for 16-bit tensors, global_load_lds_dwordx4 from addresses for fp32 ones, which may pass 4 GB;
//   * ds_read_b64_tr_b16 reads a 16 x 4 block of 16-bit values transposed: within 16 lanes, lane j receives
//     element (j % 4) of lanes j/4, j/4 + 4, j/4 + 8, j/4 + 12.  With lanes pointed at 4 rows x 4 column groups
//     of a raw slab, lane j gets four consecutive unfolded rows of column j: an MFMA operand half.
// Rows outside a workgroup's range, taps that fall into the zero padding and columns beyond the matrix lie outside the buffer, which reads as
// zeros (fp32: are fetched from a 16-byte block of zeros), so the slab in LDS is always complete and the inner loop has no special cases.
//
// What bounds it and how it is cut.  A TW x TW tile moves 2 TW elements per row through the L1 (64 bytes per cycle and
// CU) for TW^2 multiply-adds, so with 128-wide tiles the copies alone take as many cycles as the matrix cores: where there
// is enough work (takes_wide), wide matrices get 256-wide tiles (8 wavefronts of 128 x 64, a ring of four 32-row slabs), which
// halves that.  Matrices of up to 128 (64) columns get one tile of that width.
// Measured (ResNet-50, channels last, shared tap sums): batch 128, 256-wide: 1.85 TFLOP executed in 1.67 ms, matrix cores busy in 68 % of
// the cycles in which a CU holds a workgroup (53 % with the copies' addresses between the products and flat epilogues), LDS in 27 %; 128- and
// 64-wide: 31 % and 20 %.  The rest is wavefronts waiting at the slabs' barriers and a tile's epilogue, beside which a 256-wide
// workgroup has nothing else on its CU; at that load the clock falls to about 1.9 GHz.  All factors from NCHW: bf16 at batch 32
// 2090 -> 1804 us with shared sums, 1515 with planes read as they lie, 1272 with both sides of a slab's work interleaved, work dealt evenly
// to the XCDs and epilogues from 32-bit offsets; fp32 at batch 8 2555 -> 1974 -> 1766 -> 1600, and 1424 in pieces.  No vector registers live in
// scratch memory but one of the 128-wide kernel with planes (16-bit), used outside the product loops.
//
// The bias column is not part of the tiled matrix (2048 + 1 columns would cost a ninth row of 256-wide tiles for one
// column): its row of the result is the column sums, which the wavefronts of a diagonal tile whose part lies above the
// diagonal form as products with a vector of ones.
//
// Column order and padding.  Internally columns run in 16-byte vectors of V = 8 (fp32: 4) channels: (tap, channel) for
// KFAC_ORDER_KH_KW_C, (channel vector, tap, channel in vector) for KFAC_ORDER_C_KH_KW, and the channels of a tensor that
// was repacked (other layouts, channel counts that are no multiple of V) may be padded with zeros; with up to four channels
// and an even stride a vector is two neighbouring pixels instead (View::rows: the 147 columns of a 7 x 7 convolution over
// three channels become 224 instead of 392).  The epilogue puts
// results where the caller's order wants them (result_index); a vector's V kh kw columns are neighbours in both orders,
// so a tile's stores stay inside the same few cache lines.
#pragma once

#include "common.h"
#include "factor_mfma.h"

namespace kfac {

static __device__ uint4 g_zero_chunk = {0u, 0u, 0u, 0u};

typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

#define KFAC_TR_READ(dst, addr, off) \
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off))

constexpr int SHARED_ROWS_MIN = 1024, SHARED_INPUT_MIN = 1 << 17;

// A build as the matrix-core kernels see it.
struct View {
    Unfold u;        // the tensor they read: channels last, C a multiple of the 16-byte vector; d = data columns (no bias)
    int dout;        // rows of the result
    int cout;        // channels of the caller's tensor
    int chunked;     // internal column order: (channel vector, tap, channel in vector)
    int mapped;      // internal column index != result index
    int repack;      // the tensor is a repacked copy in the build's workspace
    int run;         // columns per kernel tap (C), or, if `rows`, per kernel row
    int rows;        // few channels: a repacked pixel has 4, and a kernel row's kw pixels in a row (an even number, the last one
                     // of no interest if kw is odd) are one run of columns; the copy has the zero padding in it, so that every
                     // run is whole.  The view's kw is 1, its pad 0.
    int kw;          // the layer's kernel width
    int shared;      // tap pairs at the same offset share their sums (factor_shared.h)
    int planes;      // the caller's NCHW tensor is read as it lies: a column is a channel's plane, 16 bytes are V of its rows
};

// Whether a 3 x 3 layer of stride 1 and padding 1 is built from the sums that its tap pairs share (factor_shared.h): 13 C x C
// blocks (offset (0, 0): its lower half) instead of the lower half of a 9 C x 9 C matrix, in whole tiles.  A 64-wide tile
// moves twice as many bytes per product as a 128-wide one.  At most half as many: the strips and the second launch cost something
// too.  A build's form depends on its shape alone, so that a call of few builds gives the single calls' bits.
// Time of the shared form over the dense one's, one build and 16 in a call, bf16, (tap, channel) order:
//     rows     64 channels    128            256            512
//     784      0.64  0.92     0.85  1.22     0.91  1.28     0.99  1.38
//     1176                    0.90  1.16     0.62  1.15     0.89  1.26
//     1568     0.80  0.65     0.92  1.03     0.62  1.14     0.84  1.11
//     2352                    0.87  0.53     0.58  0.95     0.74  0.92
//     3136     0.78  0.66     0.85  0.52     0.55  0.87     0.70  0.82
// ((channel, tap) order: 128 channels 0.97 and 1.08, 512 channels 1.11 and 0.90 at 1,176 rows; fp32 0.3 to 0.9 everywhere.)  The line in
// rows, 1,024, lies where a single dense build starts to need a second launch too.  From there to 2,000 rows a call of many builds of 128
// and more channels would be faster dense, by up to 30 %, whole networks of such batches (6 to 8 and 24 to 28 images) by 1 to 4 % of their
// factor builds; but dense chains of so many rows err twice as much (256 channels, 1,568 rows: 1.5e-7 against 7.6e-8; 512: 1.46e-7
// against 1.15e-7), so they are not.  The line in elements keeps 64 channels dense below 2,048 rows; the shared form is the faster one there.
static inline __host__ __device__ bool taps_shared(const Unfold& u) {
    if (u.kh != 3 || u.kw != 3 || u.stride != 1 || u.pad != 1 || u.H < 4 || u.W < 4 || u.R < SHARED_ROWS_MIN ||
        (long long)u.R * u.C < SHARED_INPUT_MIN)
        return false;
    const long long n = ceil_div(u.d, 128), m = u.C <= 64 ? 1 : ceil_div(u.C, 128);
    const long long dense = n * (n + 1) / 2 * 4, parts = u.C <= 64 ? 13 * 2 : 4 * (m * (m + 1) / 2 + 12 * m * m);
    return 2 * parts <= dense;
}

static inline __host__ __device__ bool is_plain(const Unfold& u) { return u.kh == 1 && u.kw == 1 && u.stride == 1 && u.pad == 0; }

// False: the matrix-core kernels cannot take the build.
static inline __host__ __device__ bool make_view(const Unfold& u, View* v) {
    if (u.d >= 32768) return false;                                          // byte offsets into the result fit 32 bits
    const int V = u.dtype == KFAC_F32 ? 4 : 8;
    const bool rows = u.dtype != KFAC_F32 && u.C <= 4 && u.kw > 1 && u.stride % 2 == 0;    // (even: runs start at 16-byte addresses)
    const int npx = (u.kw + 1) / 2 * 2;                                      // pixels of a run
    const int Cp = rows ? 4 : (u.C + V - 1) / V * V;
    v->u = u;
    v->u.C = Cp;
    v->u.layout = KFAC_NHWC;
    v->u.H = rows ? (u.Ho - 1) * u.stride + u.kh : u.H;
    v->u.W = rows ? ((u.Wo - 1) * u.stride + npx + 1) / 2 * 2 : u.W;
    v->u.kw = rows ? 1 : u.kw;
    v->u.pad = rows ? 0 : u.pad;
    v->run = rows ? 4 * npx : Cp;
    // (One tap: the caller's channels, of which the last vector may hold fewer than V, in the caller's order, whatever pads the copy, so
    // that results go out in vectors.  As padded columns with a map 32 rows of 1,500 took 20.2 us instead of 13.9, 3,136 of 250 24.8 and 23.4,
    // 25,088 of 37 21.0 and 19.5.)
    const bool one_tap = u.kh * u.kw == 1;
    v->u.d = one_tap ? u.C : u.kh * (rows ? 1 : u.kw) * v->run;
    v->dout = u.d;
    v->cout = u.C;
    v->kw = u.kw;
    v->rows = rows;
    v->chunked = u.order == KFAC_ORDER_C_KH_KW && u.kh * u.kw > 1;
    v->mapped = v->chunked || (Cp != u.C && !one_tap) || rows;
    v->shared = !rows && taps_shared(v->u);
    v->repack = (u.layout == KFAC_NCHW && u.H * u.W > 1) || Cp != u.C || rows;
    v->planes = 0;
    return (long long)u.N * v->u.H * v->u.W * Cp <= 0x7fffffffLL;            // 32-bit element offsets
}

// Whether the rows of an NCHW tensor at x are read as they lie (FEED_PLANES): they are its pixels, and every 16 bytes of a plane
// are aligned and of one image.  Against repacking first, all factors of ResNet-50: bf16 at batch 32 1804 -> 1515 us (1.2 GB less
// written and read again), fp32 at batch 8 1974 -> 1766 us.
static inline bool reads_planes(const Unfold& u, const void* x) {
    const int hw = u.H * u.W;
    return u.layout == KFAC_NCHW && hw > 1 && is_plain(u) && hw % (u.dtype == KFAC_F32 ? 4 : 8) == 0 && ((uintptr_t)x & 15) == 0;
}
// The view (make_view's) of such a build.
static inline __host__ __device__ void planes_view(const Unfold& u, View* v) {
    v->u = u;
    v->u.d = v->run = u.C;
    v->mapped = v->repack = 0;
    v->planes = 1;
}

// Result index of internal data column p, or -1 for a padding column.
__device__ __forceinline__ int result_index(const View& v, int p) {
    if (p >= v.u.d) return -1;
    if (!v.mapped) return p;
    if (v.rows) {
        const int ki = p / v.run, kj = (p - ki * v.run) >> 2, c = p & 3;
        if (kj >= v.kw || c >= v.cout) return -1;
        return v.chunked ? (c * v.u.kh + ki) * v.kw + kj : (ki * v.kw + kj) * v.cout + c;
    }
    const int kk = v.u.kh * v.u.kw;
    if (v.chunked) {
        const int V = v.u.dtype == KFAC_F32 ? 4 : 8;
        const int q = p / V, c = (q / kk) * V + (p - q * V), tap = q % kk;
        return c < v.cout ? c * kk + tap : -1;
    }
    const int tap = p / v.u.C, c = p - tap * v.u.C;
    return c < v.cout ? tap * v.cout + c : -1;
}

// What one thread needs to know about its 16-byte column vector.
struct ColGroup {
    bool data;    // false: beyond the matrix
    int ki, kj;   // kernel tap
    int off;      // element offset of (ki, kj, c0) relative to the patch's top-left pixel
};

__device__ __forceinline__ ColGroup decode_group(const View& v, int gcol0) {
    const Unfold& u = v.u;
    ColGroup g;
    g.ki = g.kj = g.off = 0;
    g.data = gcol0 < u.d;
    if (g.data) {
        int tap, c0;
        if (v.chunked && !v.rows) {
            const int V = u.dtype == KFAC_F32 ? 4 : 8, kk = u.kh * u.kw;
            const int q = gcol0 / V;
            c0 = (q / kk) * V;
            tap = q % kk;
        } else {
            tap = gcol0 / v.run;
            c0 = gcol0 - tap * v.run;
        }
        g.ki = tap / u.kw;
        g.kj = tap - g.ki * u.kw;
        g.off = (g.ki * u.W + g.kj) * u.C + c0;
    }
    return g;
}

// Shape of a tile: waves WM x WN of MB x NB 32 x 32 blocks, DK rows per slab, NS slabs in the ring (two panels each; a
// diagonal tile needs one panel and has a ring twice as long in the same memory).
template <int TW, int ES>
struct TileShape;
template <> struct TileShape<256, 2> { static constexpr int WM = 2, WN = 4, MB = 4, NB = 2, DK = 32, NS = 4; };
template <> struct TileShape<128, 2> { static constexpr int WM = 2, WN = 2, MB = 2, NB = 2, DK = 32, NS = 3; };
template <> struct TileShape<64, 2>  { static constexpr int WM = 2, WN = 2, MB = 1, NB = 1, DK = 64, NS = 3; };
template <> struct TileShape<128, 4> { static constexpr int WM = 2, WN = 2, MB = 2, NB = 2, DK = 16, NS = 3; };
template <> struct TileShape<64, 4>  { static constexpr int WM = 2, WN = 2, MB = 1, NB = 1, DK = 32, NS = 3; };

template <int TW, int ES> constexpr int tile_threads() { return 64 * TileShape<TW, ES>::WM * TileShape<TW, ES>::WN; }

// Where a tile's partial sums go when the rows are split: the tiles of a split one after another, then (all splits' tiles
// done) the column sums of every split.
struct Partial {
    gfloat* tiles;        // [nsplit][ntiles][tile_floats]: 32 x 32 blocks row by row (of a matrix that is one tile, only those on
                          // and below the diagonal), each as the MFMA leaves it in the registers:
                          // float 256 q + 4 lane + i is row 8 q + 4 (lane / 32) + i, column lane % 32
    gfloat* sums;         // [nsplit][tiles_dim * TW]
};

static inline __host__ __device__ int tile_floats(int tw, int ntiles) {
    const int n = tw / 32;
    return (ntiles == 1 ? n * (n + 1) / 2 : n * n) * 1024;
}

template <int TW, int ES> constexpr int tile_ring_bytes() { return TileShape<TW, ES>::NS * 2 * TileShape<TW, ES>::DK * TW * ES; }
template <int TW, int ES> constexpr int tile_lds_bytes() { return tile_ring_bytes<TW, ES>() + 4 * TW * 4; }

template <int N> struct StaticInt { static constexpr int value = N; };
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {              // f(StaticInt<0>{}) .. f(StaticInt<N - 1>{})
    if constexpr (I < N) {
        f(StaticInt<I>{});
        static_for<N, I + 1>(f);
    }
}

// The old values of a running average, 16-byte vectors of a block of 32 rows x w columns of the result, which lies in a buffer of its own
// size: a lane's byte offset and the bytes of a row, by which the passes step on in a scalar register.  A block that is not whole (they
// fetch theirs where they are written) gets an offset outside every result (d < 32768) and no steps: a step in a scalar register is not
// part of what the buffer's size is compared with, so that none may lead behind the matrix.
constexpr unsigned OUTSIDE = 0xFFFFFFF0u;
struct OldAt {
    unsigned offset, row;
};
static inline __host__ __device__ OldAt old_at(bool whole, unsigned offset, unsigned row_bytes) {
    return OldAt{whole ? offset : OUTSIDE, whole ? row_bytes : 0u};
}
// (at row, col of the tile that begins at row0, col0 of the matrix of D data columns; diag: on the diagonal, whose tiles' upper half is a
// mirror image.  Here and where it is asked, no operator that stops at the first answer: the branches cost the product loop registers.)
static inline __host__ __device__ bool block_whole(bool diag, int row0, int row, int col0, int col, int w, int D) {
    return (row0 + row + 32 <= D) & (col0 + col + w <= D) & (!diag | (row >= col + w));
}
// Row of the block row p's pass k (lane / (w / 4) further rows in it).
static inline __host__ __device__ int pass_row(int w, int p, int k) { return p * 32 + k * (64 / (w / 4)); }

// What a tile's workgroup works on.
struct TileJob {
    int I, J;
    int r_begin, r_end;
    float scale;
    bool split;              // partial sums: the tile goes to tile_dst, the column sums of a diagonal one to sums_dst
    bool lower;              // the matrix is this tile: only its blocks on and below the diagonal are kept
    gfloat *tile_dst, *sums_dst;
    int first_pixel, partner;  // FEED_WINDOW: the rectangle's first pixel, and how many pixels behind a row's pixel the one of the
                               // tile's columns lies
};

// Where the rows come from.  PATCHES: unfolded patches of any geometry.  PIXELS: a row is a pixel, all of the tensor in order.
// WINDOW: a row is a pair of pixels at a fixed offset, the first for the tile's rows, the second for its columns; the first ones
// are an Ho x Wo rectangle of each image (factor_shared.h).  PLANES: a row is a pixel of an NCHW tensor: the contraction index is
// the fast one in memory, as the MFMA wants it, and a lane's operand is one 16-byte read.
enum { FEED_PATCHES, FEED_PIXELS, FEED_WINDOW, FEED_PLANES };

// Where a copy comes from: an offset from the tensor (16-bit), or an address.
template <int ES> struct TileAddr { typedef unsigned type; };
template <> struct TileAddr<4> { typedef unsigned long long type; };

// An operand of one K step (16 rows) of a 32-column block, as it comes from LDS: 16-bit: in two pieces of two registers, or (PLANES) in one
// of four; fp32: eight floats in four pieces of two, or two of four.
template <bool PLANES, int ES> struct OperandRegs { typedef v2u type[ES]; };
template <int ES> struct OperandRegs<true, ES> { typedef v4u type[ES / 2]; };
template <int P> __device__ __forceinline__ uint4 whole_operand(const v2u (&r)[P]) { return make_uint4(r[0].x, r[0].y, r[1].x, r[1].y); }
template <int P> __device__ __forceinline__ uint4 whole_operand(const v4u (&r)[P]) { return make_uint4(r[0].x, r[0].y, r[0].z, r[0].w); }

// fp32 operands are multiplied on the bf16 matrix cores, which are 16 times as fast as the fp32 ones: x = x0 + x1 + x2, eight bits each (x0: the
// upper half of x, which no finite x takes to infinity; x1, x2 rounded, at most 2^-6 and 2^-15 of x), exactly from 2^-110 up (below, pieces
// end at bf16's last bit, 2^-133), and all products of pieces but x2 y2, which is at most 2^-31 of x y.  Errors against 64 bits, over those of
// fp32 products: 1.00 for one row, less for more (normal and ReLU'd values, up to 25,088 rows: 0.03 to 1.00; of 75 to 98 % zeros 0.80 to 1.05).  Without
// x1 y2 and x2 y1 up to 4.0 * 2^-24 of a product is lost, in a column of one value always the same way: errors of up to 8 rows, and of
// 95 % zeros, were 1.3 to 1.5 times those of fp32 products.  All factors of ResNet-50 from NCHW at batch 8: fp32 products 1616 us, six
// products of pieces 1260, these eight 1424, now 1400; six with x0 rounded (and kept finite) 1390, single products 1.02 to 1.05 times the error.
// Bound: the matrix core takes 1,024 cycles a slab of a 128-wide tile for the products and 512 for the splitting's v_dot2_f32_bf16, which run
// on it too; without them (differences, 9 more instructions to four values) 1,431 us.  Two workgroups to a CU: three leave no room for the
// small products' sums.
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
struct Pieces {
    uint4 p[3];
};
// LESS: x0 is one less in magnitude in its last bit (zero stays), for one of a product's operands.  Squares are 0, 1 or 4 modulo 8, so that sums
// of x0 x0 lie unevenly between two fp32 numbers and are rounded up or down more often, by how many there are: the diagonal of a 3x3 layer of
// 64 channels of 28 x 28, 32 images, was off by +0.8 * 2^-24 on average, of 75 % zeros by -1.2 (1.5 times the error of fp32 products); with
// a (a - 1), even and else evenly spread, by less than 0.2.
template <bool LESS>
__device__ __forceinline__ void split_pair(float a, float b, unsigned& p0, unsigned& p1, unsigned& p2) {
    // a - piece, exact, as one instruction.  ((-1, 0) and (0, -1) in registers: as a constant inside the instruction the compiler writes
    // -1.0 for both, which the hardware takes for the second.)
    unsigned minus_first = 0x0000BF80u, minus_second = 0xBF800000u;
    asm("" : "+s"(minus_first), "+s"(minus_second));
    v2bf first, second, x0;
    __builtin_memcpy(&first, &minus_first, 4);
    __builtin_memcpy(&second, &minus_second, 4);
    p0 = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
    if constexpr (LESS) {
        unsigned up, down;                                         // (neither wraps but one at +0, the other at -0: both give 0 there)
        asm("v_pk_sub_u16 %0, %1, 1 op_sel_hi:[1,0] clamp" : "=v"(up) : "v"(p0));
        asm("v_pk_sub_i16 %0, %1, 1 op_sel_hi:[1,0] clamp" : "=v"(down) : "v"(p0));
        p0 = up & down;
    }
    __builtin_memcpy(&x0, &p0, 4);
    a = __builtin_amdgcn_fdot2_f32_bf16(x0, first, a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(x0, second, b, false);
    const v2bf x1 = {(__bf16)a, (__bf16)b};
    __builtin_memcpy(&p1, &x1, 4);
    a = __builtin_amdgcn_fdot2_f32_bf16(x1, first, a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(x1, second, b, false);
    const v2bf x2 = {(__bf16)a, (__bf16)b};
    __builtin_memcpy(&p2, &x2, 4);
}
template <bool LESS>
__device__ __forceinline__ void split_words(const unsigned (&w)[8], Pieces& o) {
    unsigned q[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pair<LESS>(__uint_as_float(w[2 * i]), __uint_as_float(w[2 * i + 1]), q[0][i], q[1][i], q[2][i]);
#pragma unroll
    for (int e = 0; e < 3; ++e) o.p[e] = make_uint4(q[e][0], q[e][1], q[e][2], q[e][3]);
}
template <bool LESS>
__device__ __forceinline__ void split_operand(const v2u (&r)[4], Pieces& o) {
    const unsigned w[8] = {r[0].x, r[0].y, r[1].x, r[1].y, r[2].x, r[2].y, r[3].x, r[3].y};
    split_words<LESS>(w, o);
}
template <bool LESS>
__device__ __forceinline__ void split_operand(const v4u (&r)[2], Pieces& o) {
    const unsigned w[8] = {r[0].x, r[0].y, r[0].z, r[0].w, r[1].x, r[1].y, r[1].z, r[1].w};
    split_words<LESS>(w, o);
}
// Pieces of the eight products, smallest first.  The first seven have accumulators of their own: the matrix cores cut sums off, and all
// products to an accumulator of sums of one sign would err up to 2.5 times as much as fp32 products.
constexpr int SPLIT_PRODUCTS = 8;
constexpr int split_a(int e) { return e < 2 ? e + 1 : e < 5 ? e - 2 : e < 7 ? e - 5 : 0; }       // 1 2 0 1 2 0 1 0
constexpr int split_b(int e) { return e < 2 ? 2 - e : e < 5 ? 4 - e : e < 7 ? 6 - e : 0; }       // 2 1 2 1 0 1 0 0

// One tile.  KIND 0: bf16, 1: fp16, 2: fp32.
template <int TW, int KIND, int FEED, bool DIAG>
__device__ __forceinline__ void factor_tile_run(const View& v, const KFAC_AS1 unsigned char* x, const TileJob& job,
                                                const OutSpec& os, unsigned char* smem) {
    constexpr bool PLAIN = FEED == FEED_PIXELS, WINDOW = FEED == FEED_WINDOW, PLANES = FEED == FEED_PLANES;
    constexpr int ES = KIND == 2 ? 4 : 2, V = 16 / ES;
    typedef TileShape<TW, ES> S;
    constexpr int NW = S::WM * S::WN, DK = S::DK;
    constexpr int PANEL = DK * TW * ES;                        // bytes of one operand panel of one slab
    constexpr int STAGE = DIAG ? PANEL : 2 * PANEL;
    constexpr int NS = DIAG ? 2 * S::NS : S::NS;
    constexpr int NP = DIAG ? 1 : 2;                           // panels
    constexpr int NB2 = PANEL / 1024 / NW;                     // copies (1 KB each) per wavefront, slab and panel
    constexpr int NI = NP * NB2;
    static_assert(NB2 == 2 && NB2 * NW * 1024 == PANEL && (NS - 1) * NI < 64, "every wavefront issues two copies a panel");
    constexpr int RGS = 8 * TW;                                // 16-bit: bytes of four rows
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    const Unfold& u = v.u;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave / S::WN, wn = wave % S::WN;
    const int lm = lane & 31, h = lane >> 5;
    const int I = __builtin_amdgcn_readfirstlane(job.I), J = __builtin_amdgcn_readfirstlane(job.J), D = u.d;
    const int r_begin = __builtin_amdgcn_readfirstlane(job.r_begin), r_end = __builtin_amdgcn_readfirstlane(job.r_end);
    const int nst = (r_end - r_begin + DK - 1) / DK;
    const int wr = wm * S::MB * 32, wc = wn * S::NB * 32;      // this wavefront's part of the tile

    // ---- producer: this wavefront fills blocks block(0) and block(1) of every panel; block = 64 consecutive 16-byte slots ----
    // 16-bit slab: slot (row r, vector q) of four rows 4 rg .. 4 rg + 3 is rg (TW / 2) + 8 (q / 2) + 2 (r % 4) + q % 2: every
    // 16-lane transposed read is then a contiguous 128-byte run.  fp32 slab: row-major.
    // A lane copies the same rows of both panels: one row (two vectors of each panel) of a 256-wide slab, else two rows, so that
    // most of the address arithmetic, which runs on the pipes the matrix cores are issued from, is done once for two or four copies.
    // PLANES: slot = column CH + (16 bytes of its DK rows ^ a number that differs in any 16 columns read at once): a lane's row is
    // the same in all blocks, its column CSTEP further on from block to block.
    constexpr bool PAIR = !PLANES && TW == 256;                // both blocks hold the same four rows
    constexpr int NR = PLANES || PAIR ? 1 : 2, NC = PAIR ? 2 : 1;      // rows, and vectors of a panel's row, of a lane
    constexpr int CH = DK / V, CSTEP = NW * 64 / CH, LESS = 16 / CH;
    static_assert(CSTEP % 16 == 0, "the flip is the same in all blocks");
    auto block = [&](int j) { return PAIR ? 2 * wave + j : wave + NW * j; };
    int row0, q;                                               // row inside the slab, vector (PLANES: column) of block 0
    constexpr int ROWSTEP = ES == 4 ? NW * 64 / (TW / 4) : NW * 64 / (TW / 2) * 4;    // rows from block 0 to block 1 (not PAIR)
    {
        const int L = block(0) * 64 + lane;
        if constexpr (PLANES) {
            q = L / CH;
            row0 = ((L % CH) ^ (q / LESS % CH)) * V;
        } else if constexpr (ES == 4) {
            row0 = L / (TW / 4);
            q = L % (TW / 4);
        } else {
            const int s = L % (TW / 2);
            row0 = 4 * (L / (TW / 2)) + ((s & 7) >> 1);
            q = 2 * (s >> 3) + (s & 1);
        }
    }
    lds_byte* lds0 = (lds_byte*)smem;
    // 16-bit tensors stay below 4 GB (make_view): byte offsets of 32 bits, and what is to be zero lies outside the buffer, for which
    // the hardware gives zeros.  fp32 ones need 64 bits, and a block of zeros.
    typedef typename TileAddr<ES>::type addr_t;
    const unsigned bytes = (unsigned)(ES * ((long long)u.N * u.H * u.W * u.C));
    const __amdgpu_buffer_rsrc_t tensor = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, bytes, 0x00027000);
    const addr_t base = ES == 2 ? (addr_t)0 : (addr_t)(unsigned long long)x;
    const addr_t nowhere = ES == 2 ? (addr_t)0xFFFFFFF0u : (addr_t)(unsigned long long)(const KFAC_AS1 unsigned char*)&g_zero_chunk;
    int left = r_end - r_begin - row0;                         // the lane's (first) row is there while this is positive

    // Columns: of the lane's vectors, the byte offset behind the row's, the tap (PATCHES; never in the image if the vector lies beyond
    // the matrix), and what `left` has to exceed (the others; -> never).
    addr_t coff[NP][NC];
    int cki[NP][NC], ckj[NP][NC], need[NP][NC];
    if constexpr (!PLANES) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int col = (p == 0 ? I : J) * TW + (q + c * 16) * V;
                ColGroup g;
                if constexpr (WINDOW) {
                    g.ki = g.kj = 0;
                    g.data = col < D;
                    g.off = col + (p == 0 ? job.first_pixel : job.first_pixel + job.partner) * u.C;
                } else {
                    g = decode_group(v, col);
                }
                coff[p][c] = (addr_t)((long long)ES * g.off);
                cki[p][c] = g.data ? g.ki - u.pad : 0x40000000;
                ckj[p][c] = g.kj - u.pad;
                need[p][c] = g.data ? 0 : 0x7fffffff;
            }
    }

    // PLANES: this lane's 16 bytes of column q, advanced by DK pixels from slab to slab: pn images and pp pixels, with at most one carry.
    addr_t plane_at = 0, plane_step = 0, plane_carry = 0, plane_col[NP][2];
    int plane_px = 0, plane_dx = 0;
    if constexpr (PLANES) {
        const int size = u.H * u.W, R = r_begin + row0, n = R / size;
        plane_px = R - n * size;
        plane_dx = DK % size;
        plane_at = base + (addr_t)((long long)ES * ((long long)n * u.C * size + plane_px));
        plane_step = (addr_t)(ES * ((long long)(DK / size) * u.C * size + plane_dx));
        plane_carry = (addr_t)(ES * ((long long)u.C - 1) * size);
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int col = (p == 0 ? I : J) * TW + q + j * CSTEP;
                plane_col[p][j] = (addr_t)((long long)ES * col * size);
                need[p][0] = 0;
                if (j == 0) cki[p][0] = D - col;               // (column j: there while above j CSTEP)
            }
    }

    // The rows whose vectors this lane copies, advanced by DK rows from slab to slab without divisions: DK rows are
    // dn images, dy image rows and dx pixels, each with at most one carry into the next.
    addr_t at[NR];                                             // address of the row's patch origin
    int ty[NR], tx[NR];                                        // the patch origin's place in the (padded) image
    const int hw = u.Ho * u.Wo;
    const int dn = DK / hw, dyr = DK % hw, dy = dyr / u.Wo, dx = dyr % u.Wo;
    const long long px = (long long)ES * u.C;                  // bytes of a pixel
    const int st_x = dx * u.stride, st_y = dy * u.stride, wrap_x = u.Wo * u.stride, wrap_y = u.Ho * u.stride;
    const addr_t step_bytes = (addr_t)(PLAIN ? DK * px : px * ((long long)dn * u.H * u.W + (long long)st_y * u.W + st_x));
    const addr_t carry_x = (addr_t)(px * ((long long)u.stride * u.W - wrap_x));
    const addr_t carry_y = (addr_t)(px * ((long long)u.H * u.W - (long long)wrap_y * u.W));
    if constexpr (!PLANES) {
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int R = r_begin + row0 + j * ROWSTEP;
            if constexpr (PLAIN) {
                at[j] = base + (addr_t)((long long)R * px);
            } else {
                const int n = R / hw, rem = R - n * hw, yo = rem / u.Wo, xo = rem - yo * u.Wo;
                ty[j] = yo * u.stride;
                tx[j] = xo * u.stride;
                at[j] = base + (addr_t)(px * (((long long)n * u.H + ty[j] - u.pad) * u.W + tx[j] - u.pad));
            }
        }
    }

    // Where copy i of the next slab comes from (branch-free; slabs in order; i = 2 p + block), the step on to the slab after it, and the
    // copy itself, into the ring at stage_off.
    auto source = [&](auto i) -> addr_t {
        constexpr int p = decltype(i)::value / 2, b = decltype(i)::value % 2, j = NR == 2 ? b : 0, c = PAIR ? b : 0;
        if constexpr (PLANES) {
            return ((left > 0) & (cki[p][0] > b * CSTEP)) ? plane_at + plane_col[p][b] : nowhere;
        } else {
            bool ok;
            if constexpr (FEED == FEED_PATCHES)
                ok = (left > j * ROWSTEP) & ((unsigned)(ty[j] + cki[p][c]) < (unsigned)u.H) & ((unsigned)(tx[j] + ckj[p][c]) < (unsigned)u.W);
            else
                ok = left - j * ROWSTEP > need[p][c];
            return ok ? at[j] + coff[p][c] : nowhere;
        }
    };
    auto advance = [&]() {
        if constexpr (PLANES) {
            plane_at += plane_step;
            plane_px += plane_dx;
            const bool carry = plane_px >= u.H * u.W;
            plane_px -= carry ? u.H * u.W : 0;
            plane_at += carry ? plane_carry : 0;
        } else {
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                if constexpr (PLAIN) {
                    at[j] += step_bytes;
                } else {
                    tx[j] += st_x;
                    const bool cx = tx[j] >= wrap_x;
                    tx[j] -= cx ? wrap_x : 0;
                    ty[j] += st_y + (cx ? u.stride : 0);
                    const bool cy = ty[j] >= wrap_y;
                    ty[j] -= cy ? wrap_y : 0;
                    at[j] += step_bytes + (cx ? carry_x : 0) + (cy ? carry_y : 0);
                }
            }
        }
        left -= DK;
    };
    auto copy = [&](addr_t src, auto i, int stage_off) {
        __attribute__((address_space(3))) void* dst =
            (__attribute__((address_space(3))) void*)(lds0 + stage_off + decltype(i)::value / 2 * PANEL + block(decltype(i)::value % 2) * 1024);
        if constexpr (ES == 2)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(tensor, dst, 16, (int)src, 0, 0, 0);
        else
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, dst, 16, 0, 0);
    };

    // ---- pipeline ----
    // A slab is multiplied in STEPS steps; the operands of the next step are on their way from LDS while one is multiplied
    // (read: starts one of READS operand reads into one of two register sets; multiply: one of the MULS products of a set).  The barrier
    // sits before a slab's last step: this wavefront has then read all of the slab, so that once everybody is there the slab's place may
    // be refilled, which the next slab's first step does, and the first operands of the next slab, whose copies have landed, are read
    // during the last step's products.  A product occupies the matrix cores for 32 cycles: reads, address arithmetic and
    // copies are dealt out between the products, one fenced group after each (left alone, they gather before or behind them, in all
    // wavefronts at the same time).
    // fp32: one register set, emptied (split into pieces) before the next operands are read into it; where a slab is one step, its place is
    // free from the start of its products on, and all of the ring is filled ahead.
    constexpr int STEPS = DK / 16;
    static_assert(STEPS % 2 == 0 || ES == 4, "the register sets alternate across slabs");
    constexpr int AHEAD = STEPS == 1 ? NS : NS - 1;                                 // slabs copied before the first is read
    auto set_of = [](int step) { return ES == 2 ? step & 1 : 0; };
    auto pipeline = [&](auto muls, auto reads, auto&& read, auto&& arrived, auto&& multiply) {
        constexpr int MULS = decltype(muls)::value, READS = decltype(reads)::value;
        constexpr int SLOTS = MULS > 0 ? MULS : 1, LAST = SLOTS - SLOTS / 4;        // reads go behind the first LAST products
        constexpr int CPS = (NI + 1 + SLOTS - 1) / SLOTS;                           // copies (and the step on) to a slot
        auto step = [&](auto e, int next_off, int freed) {                          // multiply step e, read step e + 1, refill `freed`
            constexpr int E = decltype(e)::value, NEXT = (E + 1) % STEPS;
            arrived(set_of(E));
            static_for<SLOTS>([&](auto m) {
                constexpr int M = decltype(m)::value;
                if constexpr (MULS > 0) multiply(m, set_of(E));
                if constexpr (M < LAST)
                    static_for<READS * (M + 1) / LAST - READS * M / LAST>([&](auto k) {
                        read(StaticInt<READS * M / LAST + decltype(k)::value>{}, (unsigned)next_off, StaticInt<NEXT>{}, set_of(NEXT));
                    });
                if constexpr (E == 0)
                    static_for<CPS>([&](auto k) {
                        constexpr int C = M * CPS + decltype(k)::value;
                        if constexpr (C < NI) copy(source(StaticInt<C>{}), StaticInt<C>{}, freed);
                        if constexpr (C == NI) advance();
                    });
                __builtin_amdgcn_sched_barrier(0);
            });
        };
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            static_for<NI>([&](auto i) { copy(source(i), i, s * STAGE); });
            advance();
        }
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((AHEAD - 1) * NI) : "memory");
        static_for<READS>([&](auto k) { read(k, 0u, StaticInt<0>{}, 0); });
        int cur = 0, freed = (NS - 1) * STAGE;                  // ring offset of slab s, and of the place to refill
        for (int s = 0; s < nst; ++s) {
            static_for<STEPS - 1>([&](auto e) {
                asm volatile("s_waitcnt lgkmcnt(0)");
                step(e, cur, freed);
            });
            // everything of this slab is in registers, this wavefront's copies of the next one have landed (NS - 2 later slabs
            // may still be in flight), and so for everybody
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((NS - 2) * NI) : "memory");
            freed = cur;
            cur = cur + STAGE == NS * STAGE ? 0 : cur + STAGE;
            step(StaticInt<STEPS - 1>{}, cur, freed);
        }
        // trailing (all-zero) slabs must not land later, and everybody is done with the ring
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        arrived(0);                                             // (the last read's registers are not free before that wait)
    };

    // ---- consumer: LDS byte address of this lane's operand pieces in stage 0, from tile column c0 on ----
    auto operand_addr = [&](int c0) -> unsigned {
        if constexpr (PLANES) {
            return (unsigned)((c0 + lm) * CH + (h * (ES / 2) ^ (lm / LESS % CH))) * 16;
        } else if constexpr (ES == 2) {
            const int grp = lane >> 4, p = lane & 15, r = p >> 2, cg4 = p & 3;
            return (unsigned)((2 * (grp >> 1)) * RGS + (2 * r + (cg4 >> 1)) * 16 + (cg4 & 1) * 8 + (grp & 1) * 128 + c0 / 16 * 128);
        } else {
            return (unsigned)((8 * h * TW + c0 + lm) * 4);
        }
    };
    // Read k of a block's operand for the e-th K step (16 rows) of a slab: lane (lm, h) gets rows 8 h .. 8 h + 7 of the step.  16-bit: two
    // transposing reads (counted as one), PLANES: one of 16 bytes.  fp32: four reads of two rows each, PLANES: two of 16 bytes.
    constexpr int OPERAND_READS = ES == 2 ? 1 : PLANES ? 2 : 4;
    constexpr int PRODUCTS = ES == 2 ? 1 : SPLIT_PRODUCTS;     // MFMAs of a step and block
    typedef typename OperandRegs<PLANES, ES>::type Regs;
    constexpr int U = TW / 64;                                 // fp32: units of 256 bytes per slab row
#define KFAC_TILE_READ(dst, i, k, addr, step)                                                                                     \
    do {                                                                                                                         \
        if constexpr (PLANES) {                                                                                                  \
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst[k]) : "v"((addr) ^ (16u * (ES * decltype(step)::value + k))), "n"((i) * 32 * CH * 16)); \
        } else if constexpr (ES == 2) {                                                                                          \
            KFAC_TR_READ(dst[0], addr, (i) * 256 + (4 * decltype(step)::value + 0) * RGS);                                                          \
            KFAC_TR_READ(dst[1], addr, (i) * 256 + (4 * decltype(step)::value + 1) * RGS);                                                          \
        } else {                                                                                                                 \
            asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3"                                                          \
                         : "=v"(dst[k]) : "v"(addr + (i) * 128), "n"(U * (16 * decltype(step)::value + 2 * (k))), "n"(U * (16 * decltype(step)::value + 2 * (k) + 1))); \
        }                                                                                                                        \
    } while (0)
    auto operand_arrived = [](Regs& r) {
#pragma unroll
        for (int k = 0; k < (int)(sizeof(Regs) / sizeof(r[0])); ++k) asm volatile("" : "+v"(r[k]));
    };

    // A wavefront whose part lies beyond the matrix or (diagonal tile) wholly above the diagonal only takes part in the
    // copies; the latter form the column sums instead, BB 32-column blocks each.
    constexpr int BB = TW == 64 ? 2 : 4;
    constexpr int FIRST_ABOVE = S::MB / S::NB;                 // first such wavefront of wave row 0
    static_assert(S::WN - FIRST_ABOVE == TW / (BB * 32), "the wavefronts above the diagonal cover the tile's columns");
    const bool above = DIAG && wm == 0 && wn >= FIRST_ABOVE;
    const int d = v.dout;
    gfloat* __restrict__ out = os.dst;
    const bool packed = os.mode == OUT_PACKED, ema = os.mode == OUT_EMA;
    const bool split = WINDOW || job.split;
    // result row of each of the tile's rows and columns (-1: none), and the same times the result's width
    int* rmap = (int*)(smem + tile_ring_bytes<TW, ES>());
    int* cmap = rmap + TW;
    int* rmapd = rmap + 2 * TW;
    int* cmapd = rmap + 3 * TW;
    if (!split) {
        for (int e = t; e < 2 * TW; e += 64 * NW) {
            const int ri = result_index(v, e < TW ? I * TW + e : J * TW + e - TW);
            rmap[e] = ri;
            rmapd[e] = ri < 0 ? -1 : ri * d;
        }
        __syncthreads();
    }
    if (above) {
        const int c0 = (wn - FIRST_ABOVE) * BB * 32;
        if (!u.has_bias || J * TW + c0 >= D) {
            pipeline(StaticInt<0>{}, StaticInt<0>{}, [](auto, unsigned, auto, int) {}, [](int) {}, [](auto, int) {});
            return;
        }
        v16f acc[BB];
#pragma unroll
        for (int i = 0; i < BB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
        const unsigned addr0 = operand_addr(c0);
        Regs b[ES == 2 ? 2 : 1][BB];
        Pieces bp[ES == 2 ? 1 : BB];
        v16f low[ES == 2 ? 1 : BB] = {};
        pipeline(StaticInt<BB * (ES == 2 ? 1 : 3)>{}, StaticInt<BB * OPERAND_READS>{}, [&](auto k, unsigned stage_off, auto e, int set) {
            constexpr int i = decltype(k)::value / OPERAND_READS, part = decltype(k)::value % OPERAND_READS;
            KFAC_TILE_READ(b[set][i], i, part, addr0 + stage_off, e);
        }, [&](int set) {
#pragma unroll
            for (int i = 0; i < BB; ++i) operand_arrived(b[set][i]);
            if constexpr (ES == 4) {
#pragma unroll
                for (int i = 0; i < BB; ++i) split_operand<false>(b[0][i], bp[i]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }, [&](auto m, int set) {
            constexpr int i = decltype(m)::value % BB, e = decltype(m)::value / BB;
            const unsigned one2 = KIND == 1 ? 0x3C003C00u : 0x3F803F80u;
            const uint4 ones = make_uint4(one2, one2, one2, one2);
            if constexpr (ES == 2) acc[i] = mfma16<KIND == 1>(ones, whole_operand(b[set][i]), acc[i]);
            else if constexpr (e < 2) low[i] = mfma16<false>(ones, bp[i].p[2 - e], low[i]);
            else acc[i] = mfma16<false>(ones, bp[i].p[0], acc[i]);
        });
        if constexpr (ES == 4) {
#pragma unroll
            for (int i = 0; i < BB; ++i) acc[i] += low[i];
        }
        if (h == 0) {                                           // (all rows of the products are the sums)
            if (split) {
                gfloat* dst = job.sums_dst + J * TW + c0;
#pragma unroll
                for (int i = 0; i < BB; ++i) dst[i * 32 + lm] = acc[i][0];
            } else {
#pragma unroll
                for (int i = 0; i < BB; ++i) {
                    const int co = cmap[c0 + i * 32 + lm];
                    if (co >= 0) emit_sym(os, d, d - 1, co, acc[i][0] * job.scale, true);
                }
                if (J == 0 && c0 == 0 && lane == 0) emit_sym(os, d, d - 1, d - 1, (float)u.R * job.scale, false);   // R ones
            }
        }
        return;
    }
    if (I * TW + wr >= D || J * TW + wc >= D) {
        pipeline(StaticInt<0>{}, StaticInt<0>{}, [](auto, unsigned, auto, int) {}, [](int) {}, [](auto, int) {});
        return;
    }
    v16f acc[S::MB][S::NB];
#pragma unroll
    for (int i = 0; i < S::MB; ++i)
#pragma unroll
        for (int n = 0; n < S::NB; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][n][r] = 0.f;
    const unsigned a_addr = operand_addr(wr), b_addr = operand_addr(wc) + (DIAG ? 0u : (unsigned)PANEL);
    constexpr int SETS = ES == 2 ? 2 : 1;
    Regs a[SETS][S::MB], b[SETS][S::NB];
    Pieces ap[ES == 2 ? 1 : S::MB], bp[ES == 2 ? 1 : S::NB];
    v16f low[ES == 2 ? 1 : S::MB][ES == 2 ? 1 : S::NB] = {};       // the seven small products' sums (see split_a)
    pipeline(StaticInt<S::MB * S::NB * PRODUCTS>{}, StaticInt<(S::MB + S::NB) * OPERAND_READS>{}, [&](auto k, unsigned stage_off, auto e, int set) {
        constexpr int K = decltype(k)::value / OPERAND_READS, part = decltype(k)::value % OPERAND_READS;
        if constexpr (K < S::NB) KFAC_TILE_READ(b[set][K], K, part, b_addr + stage_off, e);
        else KFAC_TILE_READ(a[set][K - S::NB], K - S::NB, part, a_addr + stage_off, e);
    }, [&](int set) {
#pragma unroll
        for (int i = 0; i < S::NB; ++i) operand_arrived(b[set][i]);
#pragma unroll
        for (int i = 0; i < S::MB; ++i) operand_arrived(a[set][i]);
        if constexpr (ES == 4) {
#pragma unroll
            for (int i = 0; i < S::NB; ++i) split_operand<true>(b[0][i], bp[i]);
#pragma unroll
            for (int i = 0; i < S::MB; ++i) split_operand<false>(a[0][i], ap[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }, [&](auto m, int set) {
        constexpr int B = S::MB * S::NB, e = decltype(m)::value / B, i = decltype(m)::value % B / S::NB, n = decltype(m)::value % S::NB;
        if constexpr (ES == 2) acc[i][n] = mfma16<KIND == 1>(whole_operand(a[set][i]), whole_operand(b[set][n]), acc[i][n]);
        else if constexpr (e + 1 < PRODUCTS) low[i][n] = mfma16<false>(ap[i].p[split_a(e)], bp[n].p[split_b(e)], low[i][n]);
        else acc[i][n] = mfma16<false>(ap[i].p[0], bp[n].p[0], acc[i][n]);
    });
    if constexpr (ES == 4) {
#pragma unroll
        for (int i = 0; i < S::MB; ++i)
#pragma unroll
            for (int n = 0; n < S::NB; ++n) acc[i][n] += low[i][n];
    }

    // ---- epilogue ----
    // Stores leave a CU at four lanes per cycle, whatever a lane stores: 16-byte stores wherever four neighbours are there
    // (4-byte ones took 30 us of a tile's life).
    if (split) {                                                   // partial sums: in register order, see Partial
        gfloat* dst = job.tile_dst + (size_t)lane * 4;
#pragma unroll
        for (int p = 0; p < S::MB; ++p)
#pragma unroll
            for (int n = 0; n < S::NB; ++n) {
                const int rb = wm * S::MB + p, cb = wn * S::NB + n;
                if (DIAG && cb > rb) continue;                     // (uniform)
                gfloat* blk = dst + (DIAG && job.lower ? rb * (rb + 1) / 2 + cb : rb * (TW / 32) + cb) * 1024;
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *(KFAC_AS1 v4f*)(blk + q4 * 256) = v4f{acc[p][n][4 * q4], acc[p][n][4 * q4 + 1], acc[p][n][4 * q4 + 2], acc[p][n][4 * q4 + 3]};
            }
        return;
    }
    // One 32-row block row at a time through LDS (this wavefront's own part of it): its rows go out along result rows, then
    // its columns along the rows of the mirror image.  (From the registers the stores would need an address each, which
    // costs the product loop its registers.)
    constexpr int W = S::NB * 32, LD = W + 4;
    static_assert(NW * 32 * LD * 4 <= tile_ring_bytes<TW, ES>(), "the epilogue's staging fits the ring");
    float* epi = (float*)smem + wave * (32 * LD);
    constexpr int NV = 32 * W / 256;                               // 16-byte vectors per lane of one block row
    // A block row that is all there, below the diagonal and in the caller's column order (nearly all of a large factor's).
    auto whole = [&](int p) {
        return !v.mapped & !packed & block_whole(DIAG, I * TW, wr + p * 32, J * TW, wc, W, D);
    };
    // The others in the caller's order: a block row that the diagonal crosses or the matrix's end cuts goes out in vectors too (a matrix's
    // end falls between two of them), the diagonal block with its upper half from its lower one.  (Element by element a crossed block row
    // took 4.5 us: 32 rows of 256 columns 13.6 -> 7.5 us, all factors from NCHW fp32 1230 -> 1209.)
    auto in_vectors = [&](int p) { return !v.mapped && !packed && (D % 4 == 0 || I * TW + wr + p * 32 + 32 <= D); };
    constexpr int VPR = W / 4;                                     // vectors per row
    const int vr = lane / VPR, vc = lane % VPR * 4;                // this lane's vector of the first rows
    // Running average: the old values of block row p, fetched one block row ahead, so that a tile waits for memory once
    // and not once per block row.  (Two ahead do not fit the registers beside the accumulators.)
    v4f old[2][NV];
    // Byte offsets into the result: the lane's, and, the same in all lanes, what to add for a block row and a pass.  (Addresses of 64 bits
    // for every pass do not fit the registers beside the accumulators and the old values.)
    const unsigned out_bytes = packed ? 2u * d * (d + 1) : 4u * d * d;      // (d < 32768)
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)out, 0, out_bytes, 0x00027000);
    const unsigned ud = 4u * d;
    const unsigned direct0 = (I * TW + wr + vr) * ud + 4u * (J * TW + wc + vc);
    const unsigned mirror0 = (J * TW + wc + (lane >> 3)) * ud + 4u * (I * TW + wr + (lane & 7) * 4);
    auto direct_step = [&](int p, int k) { return pass_row(W, p, k) * ud; };
    auto mirror_step = [&](int p, int k) { return k * 8 * ud + 4u * (p * 32); };
    // (without a branch, also where the old values are not wanted)
    auto fetch_old = [&](int p, v4f (&o)[NV]) {
        const OldAt at = old_at(ema & whole(p), direct0, ud);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const v4u x = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at.offset, pass_row(W, p, k) * at.row, 0);
            __builtin_memcpy(&o[k], &x, 16);
        }
    };
    // (The step is added by the vector unit: of a 16-byte store with its step in a scalar register the third dword was now and then
    // the next vector instruction's result, in the last four lanes of 16.  The compiler keeps the two apart in this form only.)
    auto put_vector = [&](unsigned off, unsigned step, const v4f& val) {
        v4u x;
        __builtin_memcpy(&x, &val, 16);
        __builtin_amdgcn_raw_buffer_store_b128(x, rsrc, off + step, 0, 0);
    };
    // Elsewhere: element by element.  Elements that are not there (beyond the matrix, padding, the other half of a diagonal
    // tile) get an offset outside the buffer, which the hardware drops: no branches, so that many are in flight.  (One body for the mirror
    // image and the packed triangle, with && and ?: in it, was compiled to a branch around each element; it cost the forms above scalar
    // registers, too.  49 rows of a 3x3 layer of 256 channels, bf16: (channel, tap) order 18.9 -> 15.5 us, packed 15.5 -> 11.8; one of
    // 64 channels 16.4 -> 12.7 and 13.9 -> 10.2.)
    const int dc = lane % W, dr = lane / W;
    constexpr int RPP = 64 / W;                                    // rows per pass of the wavefront's lanes
    const int cod = cmap[wc + dc];
    auto direct_off = [&](int rl, int rd) -> unsigned {            // element (row rl of the tile, this lane's column)
        return rd >= 0 && cod >= 0 && !(DIAG && rl < wc + dc) ? (unsigned)(rd + cod) * 4u : ~0u;
    };
    fetch_old(0, old[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < S::MB; ++p) {
        const int rb = wr + p * 32;
        asm volatile("" ::: "memory");                             // (nothing read from the maps is kept for the next block row)
#pragma unroll
        for (int n = 0; n < S::NB; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) epi[((r >> 2) * 8 + h * 4 + (r & 3)) * LD + n * 32 + lm] = acc[p][n][r] * job.scale;
        __builtin_amdgcn_sched_barrier(0);
        if (whole(p)) {
            if (p + 1 < S::MB) fetch_old(p + 1, old[(p + 1) & 1]);
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                float* e = &epi[(k * (64 / VPR) + vr) * LD + vc];
                v4f val = *(const v4f*)e;
                if (ema) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) val[i] = fmaf(os.decay, old[p & 1][k][i], os.one_minus * val[i]);
                    *(v4f*)e = val;                                // (the mirror image gets the same new values)
                }
                put_vector(direct0, direct_step(p, k), val);
            }
            // mirror image: lane = four rows of one column, eight columns per pass
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const float* e = &epi[(lane & 7) * 4 * LD + k * 8 + (lane >> 3)];
                const v4f val = {e[0], e[LD], e[2 * LD], e[3 * LD]};
                put_vector(mirror0, mirror_step(p, k), val);
            }
            __builtin_amdgcn_sched_barrier(0);
            continue;
        }
        if (in_vectors(p)) {
            // (Worked out here and not ahead: neither the lanes' addresses nor, for all block rows, these scalars fit the registers.)
            int ln = lane, top = I * TW + rb, end = D, side = J * TW + wc;
            unsigned ud = 4u * d;
            asm volatile("" : "+v"(ln), "+s"(top), "+s"(end), "+s"(ud), "+s"(side));
            const int left = DIAG ? top - side : W;                // columns left of the diagonal block
            const int rows = min(32, end - top), cols = min(W, left + rows);
            if (left >= 0 && rows > 0) {                           // (else nothing of it is there, or all above the diagonal)
                const int xr = ln / VPR, xc = ln % VPR * 4;
                const unsigned corner = top * ud + 4u * side;
                if (ema) {                                         // (lanes beyond what is there fetch its last vectors)
#pragma unroll
                    for (int k = 0; k < NV; ++k) {
                        const v4u x = __builtin_amdgcn_raw_buffer_load_b128(
                            rsrc, corner + min(k * (64 / VPR) + xr, rows - 1) * ud + 4u * min(xc, cols - 4), 0, 0);
                        __builtin_memcpy(&old[p & 1][k], &x, 16);
                    }
#pragma unroll
                    for (int k = 0; k < NV; ++k) {
                        float* e = &epi[(k * (64 / VPR) + xr) * LD + xc];
                        v4f val = *(const v4f*)e;
#pragma unroll
                        for (int i = 0; i < 4; ++i) val[i] = fmaf(os.decay, old[p & 1][k][i], os.one_minus * val[i]);
                        *(v4f*)e = val;
                    }
                }
                const bool there = xc < cols;
                const int x0 = there ? xc : 0;
#pragma unroll 2
                for (int k = 0; k < NV; ++k) {
                    const int r = k * (64 / VPR) + xr;
                    v4f val;
#pragma unroll
                    for (int i = 0; i < 4; ++i) val[i] = epi[x0 + i > r + left ? (x0 + i - left) * LD + r + left : r * LD + x0 + i];
                    put_vector((int)there & (int)(r < rows) ? corner + r * ud + 4u * xc : OUTSIDE, 0, val);
                }
                const int mr = (ln & 7) * 4, mc = ln >> 3;
                const unsigned mirror = (side + mc) * ud + 4u * (top + mr);
#pragma unroll 2
                for (int k = 0; k < min(W, left) / 8; ++k) {
                    const float* e = &epi[mr * LD + k * 8 + mc];
                    const v4f val = {e[0], e[LD], e[2 * LD], e[3 * LD]};
                    put_vector(mr < rows ? mirror + k * 8 * ud : OUTSIDE, 0, val);
                }
            }
            if (p + 1 < S::MB) fetch_old(p + 1, old[(p + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            continue;
        }
        if (!packed) {
#pragma unroll
            for (int k0 = 0; k0 < 32 / RPP; k0 += 16) {
                int rd[16];
                float val[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    rd[k] = rmapd[rb + (k0 + k) * RPP + dr];
                    val[k] = epi[((k0 + k) * RPP + dr) * LD + dc];
                }
                if (ema) {
                    float o[16];
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        o[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, direct_off(rb + (k0 + k) * RPP + dr, rd[k]), 0, 0));
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        val[k] = fmaf(os.decay, o[k], os.one_minus * val[k]);
                        epi[((k0 + k) * RPP + dr) * LD + dc] = val[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val[k]), rsrc, direct_off(rb + (k0 + k) * RPP + dr, rd[k]), 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // the mirror image, or the packed triangle
        int ln = lane;
        asm volatile("" : "+v"(ln));                               // (what the block rows have in common is worked out for each)
        const int row = rb + (ln & 31), first = wc + (ln >> 5), ro = rmap[row];
        const float* from = &epi[(ln & 31) * LD + (ln >> 5)];
        auto columns = [&](auto is_packed) __attribute__((always_inline)) {
            constexpr bool PACKED = decltype(is_packed)::value;
#pragma unroll 1
            for (int c0 = 0; c0 < W; c0 += 32) {
                int cd[16];
                float val[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    cd[k] = (PACKED ? cmap : cmapd)[first + c0 + 2 * k];
                    val[k] = from[c0 + 2 * k];
                }
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const bool ok = (ro >= 0) & (cd[k] >= 0) & (!DIAG | (row >= first + c0 + 2 * k + !PACKED));
                    const unsigned e = PACKED ? (unsigned)(packed_row_base(min(ro, cd[k]), d) + max(ro, cd[k])) : (unsigned)(cd[k] + ro);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val[k]), rsrc, ok ? e * 4u : ~0u, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (packed) columns(StaticInt<1>{});
        else columns(StaticInt<0>{});
        if (p + 1 < S::MB) fetch_old(p + 1, old[(p + 1) & 1]);         // (here the registers hold no more before)
    }
}

// How a build's work list is dealt to the 8 XCDs, each with an L2 of its own.  Workgroups go to them round-robin; the caller pads every
// build's workgroup count to a multiple of 8 and starts it at a multiple of 8, so that wg % 8 is the XCD this workgroup runs on.
// XCD x takes a contiguous share of the list (row ranges in order, tiles in blocked order inside a range): the tiles of a row range,
// which all read the same rows, share one L2 instead of fetching them eight times.  `work` % 8 XCDs, from XCD `turn` on, get one
// more than the others; the next build's extra ones begin where this one's end (next_turn), so that a launch of many builds loads all
// XCDs alike.  (With the extra ones always from XCD 0 on, and whole eighths rounded up, its CUs held a workgroup in 68 % of the
// cycles: all factors of ResNet-50 from NCHW.)  Index in the list, or -1: a padding workgroup.
static inline __host__ __device__ int next_turn(int turn, int work) { return (turn + work) & 7; }
static inline __host__ __device__ int unit_of(int work, int wg, int turn) {
    const int y = ((wg & 7) - turn) & 7, in = wg >> 3, each = work >> 3, extra = work & 7;
    return in < each + (y < extra) ? y * each + (y < extra ? y : extra) + in : -1;
}

// One tile (workgroup `wg` of ntiles * nsplit, padded to a multiple of 8) of one factor build.
template <int TW, int KIND, bool PLANES>
__device__ __forceinline__ void factor_tile(const View& v, const KFAC_AS1 unsigned char* x, float scale, const OutSpec& os,
                                            const Partial& part, int rows_per_split, int tiles_dim, int ntiles, int nsplit,
                                            int wg, int turn, unsigned char* smem) {
    TileJob job;
    int tile, sp;
    {
        const int unit = unit_of(ntiles * nsplit, wg, turn);
        if (unit < 0) return;                                      // (uniform, before any barrier)
        sp = unit / ntiles;
        tile = unit - sp * ntiles;
    }
    tri_decode_blocked<4>(tiles_dim, tile, job.I, job.J);          // (tiles that share row panels run together: see the function)
    job.r_begin = sp * rows_per_split;
    job.r_end = min(v.u.R, job.r_begin + rows_per_split);
    job.split = nsplit > 1;
    job.lower = ntiles == 1;
    job.tile_dst = part.tiles + ((size_t)sp * ntiles + tile) * tile_floats(TW, ntiles);
    job.sums_dst = part.sums + (size_t)sp * (tiles_dim * TW);
    job.scale = scale;
    job.first_pixel = job.partner = 0;
    const bool plain = is_plain(v.u);
    if (job.I == job.J) {
        if (PLANES && v.planes) factor_tile_run<TW, KIND, PLANES ? FEED_PLANES : FEED_PIXELS, true>(v, x, job, os, smem);
        else if (plain) factor_tile_run<TW, KIND, FEED_PIXELS, true>(v, x, job, os, smem);
        else factor_tile_run<TW, KIND, FEED_PATCHES, true>(v, x, job, os, smem);
    } else if constexpr (TW > 64) {                                // (64-wide matrices are one tile)
        if (PLANES && v.planes) factor_tile_run<TW, KIND, PLANES ? FEED_PLANES : FEED_PIXELS, false>(v, x, job, os, smem);
        else if (plain) factor_tile_run<TW, KIND, FEED_PIXELS, false>(v, x, job, os, smem);
        else factor_tile_run<TW, KIND, FEED_PATCHES, false>(v, x, job, os, smem);
    }
}

}  // namespace kfac
