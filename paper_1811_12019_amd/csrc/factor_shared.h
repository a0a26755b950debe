// 3 x 3 convolutions of stride 1 and padding 1: tap pairs at the same offset share their sums.
//
// An entry of the factor, A[(t1, c1), (t2, c2)] = sum over output pixels p of x[p + t1, c1] x[p + t2, c2], depends on the taps
// only through their offset d = t2 - t1, but for the pixels at the image's edge: with q = p + t1 it is the sum over q of
// x[q, c1] x[q + d, c2], q running over those pixels for which p and q + d lie in the image.  Of the 81 tap pairs 25 offsets
// are different, and 13 of them up to a transposition.  Along an axis, an offset of 1 or 2 leaves all its pairs the same
// range; an offset of 0 leaves three (the tap before the centre never meets the last row, the one behind it never the
// first).  So the sums are formed once per offset, for axes of offset 0 in three parts (first row or column, the middle, last),
// and every tap pair adds up the parts it meets: only additions, of the same products as the dense form, 13 C x C blocks and
// their strips instead of 40.5 of them, over fewer pixels.  Products with the zero padding are not formed.
//
// Two launches: the tile kernel forms the parts (window_of; pixels of a rectangle are its rows, and no tap ever leaves the
// image, so that the copies need no checks), then factor_tile_reduce_kernel or factor_channels_kernel adds them up and writes the factor.
// Bound: the tiles as in factor_tile.h, the second launch HBM (the factor itself: 6 bytes an element).
// Measured, one layer's factor folded into its running average, bf16, channels last, against the dense form: at 32 images 64
// channels of 56 x 56 pixels 90 -> 50 us, 128 of 28 x 28 92 -> 47, 256 of 14 x 14 99 -> 45, 512 of 7 x 7 76 -> 61 (26 of
// them the tiles, 40 the second launch: 3.9 TB/s); at 128 images 292 -> 127, 243 -> 87, 245 -> 80, 224 -> 97; fp32 at 32
// images 522 -> 165, 387 -> 139, 389 -> 125, 365 -> 145.  All factors of ResNet-50, bf16: batch 32 1470 -> 1250 us, batch 128
// 4990 -> 3310 us; fp32 NCHW at batch 8 2610 -> 2010 us.
#pragma once

#include "factor_tile.h"

namespace kfac {

// Parts in four classes: 0 the 13 offsets' middles, 1 first and last rows (offsets (0, 0), (0, 1), (0, 2)), 2 first and last
// columns (offsets (0, 0), (1, 0), (2, 0)), 3 corners (offset (0, 0)).  Offset (0, 0) is symmetric: its tiles on and below the
// diagonal only.
struct SharedPlan {
    int tw, T, ntl, nf;        // tile width, tiles per dimension, lower tiles, all tiles
    int per[4];                // tiles of a split, per class
    int ns[4];                 // splits
    int first[5];              // first unit (tile of a split) of each class
    int rows;                  // rows of a workgroup, about (the longest)
    size_t ws_bytes;
};

struct Window {
    int dy, dx;                // offset
    int y0, x0, hy, wx;        // rectangle of the pixels q
};

static inline __host__ __device__ void axis_window(int d, int strip, int n, int* o, int* len) {   // strip: 0 first, 1 middle, 2 last
    if (d == 0) {
        *o = strip == 0 ? 0 : strip == 1 ? 1 : n - 1;
        *len = strip == 1 ? n - 2 : 1;
    } else {
        *o = d > 0 ? 0 : -d;
        *len = n - (d > 0 ? d : -d);
    }
}

// Offset o of 13: (0,0) (0,1) (0,2) (1,-2) .. (1,2) (2,-2) .. (2,2)
static inline __host__ __device__ int offset_dy(int o) { return o < 3 ? 0 : o < 8 ? 1 : 2; }
static inline __host__ __device__ int offset_dx(int o) { return o < 3 ? o : o < 8 ? o - 5 : o - 10; }
static inline __host__ __device__ int offset_index(int dy, int dx) { return dy == 0 ? dx : dy == 1 ? dx + 5 : dx + 10; }

static inline __host__ __device__ Window window_of(int H, int W, int cls, int member) {
    Window w;
    int ys = 1, xs = 1;
    if (cls == 0) {
        w.dy = offset_dy(member);
        w.dx = offset_dx(member);
    } else if (cls == 1) {
        w.dy = 0;
        w.dx = member >> 1;
        ys = member & 1 ? 2 : 0;
    } else if (cls == 2) {
        w.dy = member >> 1;
        w.dx = 0;
        xs = member & 1 ? 2 : 0;
    } else {
        w.dy = w.dx = 0;
        ys = member >> 1 ? 2 : 0;
        xs = member & 1 ? 2 : 0;
    }
    axis_window(w.dy, ys, H, &w.y0, &w.hy);
    axis_window(w.dx, xs, W, &w.x0, &w.wx);
    return w;
}

// The part that holds offset (dy, dx), dy > 0 or dy = 0 and dx >= 0, in strips ys, xs (of axes with offset 0).
static inline __host__ __device__ void part_of(int dy, int dx, int ys, int xs, int* cls, int* member) {
    const bool ye = dy == 0 && ys != 1, xe = dx == 0 && xs != 1;
    if (ye && xe) { *cls = 3; *member = ys + (xs >> 1); }
    else if (ye) { *cls = 1; *member = 2 * dx + (ys >> 1); }
    else if (xe) { *cls = 2; *member = 2 * dy + (xs >> 1); }
    else { *cls = 0; *member = offset_index(dy, dx); }
}

static inline __host__ __device__ bool member_symmetric(int cls, int member) { return cls == 3 || (cls == 0 ? member == 0 : member < 2); }

// (One of four plan values: taken out of the plan first, all of them.  Left to itself the compiler chooses between their addresses, and
// the plan goes to scratch memory.)
__device__ __forceinline__ int of_class(int cls, int v0, int v1, int v2, int v3) {
    const int a = uniform(v0), b = uniform(v1), c = uniform(v2), d = uniform(v3);
    return cls == 0 ? a : cls == 1 ? b : cls == 2 ? c : d;
}

// Unit of (class, member, split 0, tile 0); splits are per[cls] units apart.
__device__ __forceinline__ int shared_unit(const SharedPlan& p, int cls, int member) {
    const int sym = cls == 0 ? 1 : cls == 3 ? 4 : 2;
    return of_class(cls, p.first[0], p.first[1], p.first[2], p.first[3]) + (member < sym ? member * p.ntl : sym * p.ntl + (member - sym) * p.nf);
}

static inline __host__ __device__ int shared_workgroups(const SharedPlan& p) {
    return (p.first[1] + 7) / 8 * 8 + (p.first[4] - p.first[1] + 7) / 8 * 8;
}

// The workspace: the units' tiles (Partial's order inside a tile), then the column sums of offset (0, 0)'s nine parts.
static inline __host__ __device__ size_t shared_sums_at(const SharedPlan& p) { return (size_t)p.first[4] * p.tw * p.tw; }

__device__ __forceinline__ int splits_of(const SharedPlan& p, int cls) { return of_class(cls, p.ns[0], p.ns[1], p.ns[2], p.ns[3]); }
__device__ __forceinline__ size_t split_stride(const SharedPlan& p, int cls) {
    return (size_t)of_class(cls, p.per[0], p.per[1], p.per[2], p.per[3]) * p.tw * p.tw;
}

// One tile of one part: workgroup `wg` of shared_workgroups.
template <int TW, int KIND>
__device__ __forceinline__ void shared_tile(const View& v, const KFAC_AS1 unsigned char* x, const SharedPlan& p, gfloat* ws, int wg,
                                            int turn, unsigned char* smem) {
    // The middles (long) and the strips (short) are dealt to the XCDs apart (unit_of), so that every XCD gets its share of both.
    int base = 0, work = p.first[1];
    const int mid_wgs = (work + 7) >> 3 << 3;
    if (wg >= mid_wgs) {
        wg -= mid_wgs;
        base = work;
        turn = next_turn(turn, work);
        work = p.first[4] - work;
    }
    const int in = unit_of(work, wg, turn);
    if (in < 0) return;                                             // (uniform, before any barrier)
    const int unit = base + in;
    const int cls = unit < p.first[1] ? 0 : unit < p.first[2] ? 1 : unit < p.first[3] ? 2 : 3;
    const int sym = cls == 0 ? 1 : cls == 3 ? 4 : 2;
    // (not through of_class: with it 180 registers of the 128-wide kernel's epilogues went to scratch memory)
    const int ns = cls == 0 ? p.ns[0] : cls == 1 ? p.ns[1] : cls == 2 ? p.ns[2] : p.ns[3];
    const int per = cls == 0 ? p.per[0] : cls == 3 ? p.per[3] : p.per[1];
    const int at = unit - (cls == 0 ? 0 : cls == 1 ? p.first[1] : cls == 2 ? p.first[2] : p.first[3]);
    const int split = at / per, idx = at - split * per;
    TileJob job;
    int member;
    if (idx < sym * p.ntl) {
        member = idx / p.ntl;
        tri_decode(idx - member * p.ntl, job.I, job.J);
    } else {
        const int e = idx - sym * p.ntl;
        member = sym + e / p.nf;
        const int tile = e % p.nf;
        job.I = tile / p.T;
        job.J = tile - job.I * p.T;
    }
    const Window w = window_of(v.u.H, v.u.W, cls, member);
    View vw = v;
    vw.u.Ho = w.hy;
    vw.u.Wo = w.wx;
    vw.u.pad = 0;
    vw.u.R = v.u.N * w.hy * w.wx;
    vw.u.d = v.u.C;
    const int rows_per = ((vw.u.R + ns - 1) / ns + 63) / 64 * 64;
    job.r_begin = split * rows_per;
    job.r_end = min(vw.u.R, job.r_begin + rows_per);
    if (job.r_end < job.r_begin) job.r_begin = job.r_end;           // (rounding up may leave the last split empty: it stores zeros)
    job.split = true;
    job.lower = false;
    job.scale = 1.f;
    job.tile_dst = ws + (size_t)unit * (TW * TW);
    job.first_pixel = w.y0 * v.u.W + w.x0;
    job.partner = w.dy * v.u.W + w.dx;
    if (member_symmetric(cls, member) && job.I == job.J) {
        const int part = (cls == 0 ? 4 : cls == 1 ? (member ? 7 : 1) : cls == 2 ? (member ? 5 : 3) : (member >> 1) * 6 + (member & 1) * 2);
        job.sums_dst = ws + shared_sums_at(p) + ((size_t)part * p.ns[0] + split) * (p.T * TW);
        factor_tile_run<TW, KIND, FEED_WINDOW, true>(vw, x, job, OutSpec{}, smem);
    } else {
        job.sums_dst = nullptr;
        factor_tile_run<TW, KIND, FEED_WINDOW, false>(vw, x, job, OutSpec{}, smem);
    }
}

// ---- second launch: the factor from its parts ------------------------------------------------------------------------
constexpr int SH_REGION_LD = 33;
constexpr int SH_CB = 8, SH_EDGE = 9 * SH_CB;                       // (c, kh, kw) order: channels of a block, result rows of it
constexpr int SH_VLD = SH_CB * SH_CB + 1, SH_OLD = SH_EDGE + 1;
constexpr int SH_BLOCK_FLOATS = 3 * 32 * SH_REGION_LD;
constexpr int SH_CHANNEL_FLOATS = 49 * SH_VLD > SH_EDGE * SH_OLD ? 49 * SH_VLD : SH_EDGE * SH_OLD;

static inline __host__ __device__ int shared_assemble_wgs(const View& v) {
    const int bias = v.u.has_bias ? ceil_div(v.dout, 256) : 0;
    if (v.chunked) {
        const int nb = ceil_div(v.cout, SH_CB);
        return nb * (nb + 1) / 2 + bias;
    }
    const int cb = ceil_div(v.cout, 32);
    return cb * (cb + 1) / 2 + 12 * cb * cb + bias;
}

// Sum over the splits of this thread's four floats, `s` being the first split's (loaded ahead, with other parts').
__device__ __forceinline__ v4f sum_splits(v4f s, const gfloat* src, size_t stride, int ns) {
    int sp = 1;
    for (; sp + 4 <= ns; sp += 4) {
        v4f p[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = *(const KFAC_AS1 v4f*)(src + (size_t)(sp + k) * stride);
        s += (p[0] + p[1]) + (p[2] + p[3]);
    }
    for (; sp < ns; ++sp) s += *(const KFAC_AS1 v4f*)(src + (size_t)sp * stride);
    return s;
}

// First float of the 32 x 32 block (bi, bj) of a part, split 0.
__device__ __forceinline__ const gfloat* part_block(const SharedPlan& p, const gfloat* ws, int cls, int member, int bi, int bj) {
    const int SB = p.tw / 32, ti = bi / SB, tj = bj / SB;
    const int tile = member_symmetric(cls, member) ? ti * (ti + 1) / 2 + tj : ti * p.T + tj;
    return ws + (size_t)(shared_unit(p, cls, member) + tile) * (p.tw * p.tw) + ((bi - ti * SB) * SB + bj - tj * SB) * 1024;
}

// Stores of four neighbouring elements starting at dst, `n` of them there (from element `from` on).
__device__ __forceinline__ void store4(gfloat* dst, v4f val, int from, int n) {
    if (from <= 0 && n >= 4) {
        *(KFAC_AS1 v4f_a4*)dst = val;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i >= from && i < n) dst[i] = val[i];
    }
}

// (tap, channel) order: all tap pairs of one offset, a 32 x 32 block of channels.  The result's lower side is in the rows of the
// second tap and channel c2 (offset (0, 0): c1): one thread holds four neighbours of one row.
template <bool Y0, bool X0>
__device__ __forceinline__ void assemble_block(const View& v, const SharedPlan& p, const gfloat* ws, const OutSpec& os, float scale,
                                               int dy, int dx, int bi, int bj, float* lds) {
    constexpr int NY = Y0 ? 3 : 1, NX = X0 ? 3 : 1, NP = NY * NX;
    constexpr bool SYM = Y0 && X0;
    const int t = threadIdx.x, lr = t >> 3, lc = (t & 7) * 4, C = v.cout, d = v.dout;
    const int rb = SYM ? bi : bj, cb = SYM ? bj : bi;               // channel blocks of the lower side's rows and columns
    const int rc = rb * 32 + lr, cc = cb * 32 + lc;
    const bool diag = SYM && bi == bj;
    const bool packed = os.mode == OUT_PACKED, ema = os.mode == OUT_EMA;
    const int nlow = rc < C ? min(C - cc, diag ? lr - lc + 1 : 4) : 0;      // elements of this thread that are there
    auto pair_ok = [&](int ty, int tx) { return (unsigned)(ty + dy) < 3u && (unsigned)(tx + dx) < 3u; };
    auto low_at = [&](int ty, int tx) -> size_t {
        return (size_t)((SYM ? ty * 3 + tx : (ty + dy) * 3 + tx + dx) * C + rc) * d + (ty * 3 + tx) * C + cc;
    };
    // The old values of one tap row's pairs, a row ahead of their use: the first are in flight while the parts are added up.
    v4f old[2][3];
    auto fetch_old = [&](int ty) {
        if (!ema) return;
#pragma unroll
        for (int tx = 0; tx < 3; ++tx) {
            v4f& o = old[ty & 1][tx];
            o = v4f{0.f, 0.f, 0.f, 0.f};
            if (!pair_ok(ty, tx)) continue;
            const gfloat* from = os.dst + low_at(ty, tx);
            if (nlow >= 4) {
                o = *(const KFAC_AS1 v4f_a4*)from;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (i < nlow) o[i] = from[i];
            }
        }
    };
    fetch_old(0);
    // Parts, brought from the matrix cores' order (Partial) to rows.
    v4f S[NY][NX];
    const gfloat* src[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        int cls, member;
        part_of(dy, dx, Y0 ? k / NX : 1, X0 ? k % NX : 1, &cls, &member);
        src[k] = part_block(p, ws, cls, member, bi, bj) + t * 4;
        S[k / NX][k % NX] = *(const KFAC_AS1 v4f*)src[k];
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        int cls, member;
        part_of(dy, dx, Y0 ? k / NX : 1, X0 ? k % NX : 1, &cls, &member);
        S[k / NX][k % NX] = sum_splits(S[k / NX][k % NX], src[k], split_stride(p, cls), splits_of(p, cls));
    }
    constexpr int NL = NP < 3 ? NP : 3;                             // as many at a time as there is LDS for
#pragma unroll
    for (int k0 = 0; k0 < NP; k0 += NL) {
        const int q = t >> 6, lane = t & 63;
#pragma unroll
        for (int k = 0; k < NL; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                lds[k * (32 * SH_REGION_LD) + (8 * q + 4 * (lane >> 5) + i) * SH_REGION_LD + (lane & 31)] = S[(k0 + k) / NX][(k0 + k) % NX][i];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NL; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                S[(k0 + k) / NX][(k0 + k) % NX][i] =
                    lds[k * (32 * SH_REGION_LD) + (SYM ? lr * SH_REGION_LD + lc + i : (lc + i) * SH_REGION_LD + lr)];
        __syncthreads();
    }
    // What the taps before, at and behind the centre meet of an axis of offset 0.
    auto three = [](v4f a, v4f b, v4f c, int t3) -> v4f { return t3 == 0 ? a + b : t3 == 1 ? (a + b) + c : b + c; };
    int buf = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int ty = k / 3, tx = k % 3;
        if (tx == 0 && ty < 2) fetch_old(ty + 1);
        if (!pair_ok(ty, tx)) continue;                             // (uniform)
        v4f row[NY];
#pragma unroll
        for (int y = 0; y < NY; ++y) {
            if constexpr (X0) row[y] = three(S[y][0], S[y][1], S[y][2], tx);
            else row[y] = S[y][0];
        }
        v4f val;
        if constexpr (Y0) val = three(row[0], row[1], row[2], ty);
        else val = row[0];
        val *= scale;
        if (ema) {
#pragma unroll
            for (int i = 0; i < 4; ++i) val[i] = fmaf(os.decay, old[ty & 1][tx][i], os.one_minus * val[i]);
        }
        if (!packed) store4(os.dst + low_at(ty, tx), val, 0, nlow);
        float* tr = lds + buf * (32 * SH_REGION_LD);
        buf ^= 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) tr[lr * SH_REGION_LD + lc + i] = val[i];
        __syncthreads();
        // mirror image: row cb * 32 + lr, columns rb * 32 + lc ..
        const int mr = cb * 32 + lr, mc = rb * 32 + lc;
        if (mr < C) {
            const v4f m = {tr[lc * SH_REGION_LD + lr], tr[(lc + 1) * SH_REGION_LD + lr], tr[(lc + 2) * SH_REGION_LD + lr], tr[(lc + 3) * SH_REGION_LD + lr]};
            const int row_i = (ty * 3 + tx) * C + mr, col_i = (SYM ? ty * 3 + tx : (ty + dy) * 3 + tx + dx) * C + mc;
            const size_t dst = packed ? packed_row_base(row_i, d) + col_i : (size_t)row_i * d + col_i;
            store4(os.dst + dst, m, diag ? lr - lc + (packed ? 0 : 1) : 0, C - mc);
        }
    }
}

// (channel, tap) order: all 81 tap pairs of an 8 x 8 block of channels, which are neighbours in the result.  The 49 distinct sums
// of an element pair (7 kinds a axis: offset 0 in three parts, 1, 2, -1, -2) lie in LDS and every entry picks its own.
__device__ __forceinline__ void assemble_channel_block(const View& v, const SharedPlan& p, const gfloat* ws, const OutSpec& os, float scale,
                                                       int bi, int bj, float* lds) {
    const int t = threadIdx.x, C = v.cout, d = v.dout;
    const bool packed = os.mode == OUT_PACKED, ema = os.mode == OUT_EMA;
    constexpr int NE = (SH_EDGE * SH_EDGE + 255) / 256;
    auto there = [&](int e, int& row, int& col) -> bool {            // element e of the block's lower side: result row and column
        const int r = e / SH_EDGE, c = e - r * SH_EDGE;
        row = bi * SH_EDGE + r;
        col = bj * SH_EDGE + c;
        return e < SH_EDGE * SH_EDGE && row < 9 * C && col <= row;
    };
    float val[NE];                                                   // old values, then new ones
    if (ema) {
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            int row, col;
            const bool ok = there(t + 256 * k, row, col);
            val[k] = os.dst[ok ? (size_t)row * d + col : 0];         // (clamped, not guarded: all loads go out together)
        }
    }
    float* V = lds;
    float* O = lds;                                                  // (after V)
    constexpr int NT = (49 * 16 + 255) / 256;                        // tasks of four floats per thread
    const gfloat* src[NT];
    v4f S[NT];
    auto task_of = [&](int k, int& e, bool& turned, int& cls) {
        const int task = min(t + 256 * k, 49 * 16 - 1), l = task & 15;
        e = task >> 4;
        const int yc = e / 7, xc = e - yc * 7;
        int dy = yc < 3 ? 0 : yc < 5 ? yc - 2 : 4 - yc, dx = xc < 3 ? 0 : xc < 5 ? xc - 2 : 4 - xc, member;
        turned = dy < 0 || (dy == 0 && dx < 0);                      // held as the transposed sum of the opposite offset
        part_of(turned ? -dy : dy, turned ? -dx : dx, yc < 3 ? yc : 1, xc < 3 ? xc : 1, &cls, &member);
        const int br = turned ? bj : bi, bc = turned ? bi : bj;
        return part_block(p, ws, cls, member, br >> 2, bc >> 2) + (br & 3) * 256 + ((l >> 3) * 32 + (bc & 3) * 8 + (l & 7)) * 4;
    };
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        int e, cls;
        bool turned;
        src[k] = task_of(k, e, turned, cls);
        S[k] = *(const KFAC_AS1 v4f*)src[k];
    }
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        int e, cls;
        bool turned;
        task_of(k, e, turned, cls);
        const v4f s = sum_splits(S[k], src[k], split_stride(p, cls), splits_of(p, cls));
        const int l = t & 15, half = l >> 3, cc = l & 7;
        if (t + 256 * k < 49 * 16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) V[e * SH_VLD + (turned ? cc * 8 + half * 4 + i : (half * 4 + i) * 8 + cc)] = s[i];
        }
    }
    __syncthreads();
    // what the taps before, at and behind the centre meet: along x, then along y
    for (int task = t; task < 7 * 64; task += 256) {
        float* q = V + (task >> 6) * 7 * SH_VLD + (task & 63);
        const float a = q[0], b = q[SH_VLD], c = q[2 * SH_VLD];
        q[0] = a + b;
        q[SH_VLD] = (a + b) + c;
        q[2 * SH_VLD] = b + c;
    }
    __syncthreads();
    for (int task = t; task < 7 * 64; task += 256) {
        float* q = V + (task >> 6) * SH_VLD + (task & 63);
        const float a = q[0], b = q[7 * SH_VLD], c = q[14 * SH_VLD];
        q[0] = a + b;
        q[7 * SH_VLD] = (a + b) + c;
        q[14 * SH_VLD] = b + c;
    }
    __syncthreads();
    auto kind = [](int t1, int t2) -> int { return t1 == t2 ? t1 : t2 > t1 ? t2 - t1 + 2 : t1 - t2 + 4; };
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = min(t + 256 * k, SH_EDGE * SH_EDGE - 1), r = e / SH_EDGE, c = e - r * SH_EDGE;
        const int c1 = r / 9, t1 = r - 9 * c1, c2 = c / 9, t2 = c - 9 * c2;
        const float fresh = V[(kind(t1 / 3, t2 / 3) * 7 + kind(t1 % 3, t2 % 3)) * SH_VLD + c1 * 8 + c2] * scale;
        val[k] = ema ? fmaf(os.decay, val[k], os.one_minus * fresh) : fresh;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = t + 256 * k;
        int row, col;
        if (!there(e, row, col)) continue;
        const int r = e / SH_EDGE, c = e - r * SH_EDGE;
        if (!packed) os.dst[(size_t)row * d + col] = val[k];
        O[r * SH_OLD + c] = val[k];
    }
    __syncthreads();
    for (int e = t; e < SH_EDGE * SH_EDGE; e += 256) {
        const int r = e / SH_EDGE, c = e - r * SH_EDGE;              // mirror image: row bj .. + r, column bi .. + c
        const int row = bj * SH_EDGE + r, col = bi * SH_EDGE + c;
        if (row >= 9 * C || col >= 9 * C || (packed ? col < row : col <= row)) continue;
        os.dst[packed ? packed_row_base(row, d) + col : (size_t)row * d + col] = O[c * SH_OLD + r];
    }
}

// Bias row: the column sums of the parts that a tap meets.
__device__ __forceinline__ void assemble_bias(const View& v, const SharedPlan& p, const gfloat* ws, const OutSpec& os, float scale, int j) {
    const int C = v.cout, d = v.dout;
    if (j == 0) emit_sym(os, d, d - 1, d - 1, (float)v.u.R * scale, false);
    if (j >= 9 * C) return;
    const int tap = v.chunked ? j % 9 : j / C, c = v.chunked ? j / 9 : j - tap * C;
    const int ty = tap / 3, tx = tap - 3 * ty;
    const gfloat* sums = ws + shared_sums_at(p) + c;
    const size_t ld = (size_t)p.T * p.tw;
    float s = 0.f;
#pragma unroll
    for (int part = 0; part < 9; ++part) {
        const int y = part / 3, x = part % 3;
        if (y - ty == 2 || ty - y == 2 || x - tx == 2 || tx - x == 2) continue;
        const int ns = y == 1 ? (x == 1 ? p.ns[0] : p.ns[2]) : x == 1 ? p.ns[1] : p.ns[3];
        float q = 0.f;
        for (int sp = 0; sp < ns; ++sp) q += sums[((size_t)part * p.ns[0] + sp) * ld];
        s += q;
    }
    emit_sym(os, d, d - 1, j, s * scale, true);
}

__device__ __forceinline__ void assemble_channels(const View& v, const SharedPlan& p, const gfloat* ws, const OutSpec& os, float scale, int wg,
                                                  float* lds) {
    const int nb = ceil_div(v.cout, SH_CB), blocks = nb * (nb + 1) / 2;
    if (wg >= blocks) return assemble_bias(v, p, ws, os, scale, (wg - blocks) * 256 + (int)threadIdx.x);
    int bi, bj;
    tri_decode(wg, bi, bj);
    assemble_channel_block(v, p, ws, os, scale, bi, bj, lds);
}

__device__ __forceinline__ void assemble_blocks(const View& v, const SharedPlan& p, const gfloat* ws, const OutSpec& os, float scale, int wg,
                                                float* lds) {
    const int cb = ceil_div(v.cout, 32), low = cb * (cb + 1) / 2, blocks = low + 12 * cb * cb;
    if (wg >= blocks) return assemble_bias(v, p, ws, os, scale, (wg - blocks) * 256 + (int)threadIdx.x);
    if (wg < low) {
        int bi, bj;
        tri_decode(wg, bi, bj);
        return assemble_block<true, true>(v, p, ws, os, scale, 0, 0, bi, bj, lds);
    }
    const int e = wg - low, o = 1 + e / (cb * cb), b = e % (cb * cb), bi = b / cb, bj = b - bi * cb;
    const int dy = offset_dy(o), dx = offset_dx(o);
    if (dy == 0) assemble_block<true, false>(v, p, ws, os, scale, 0, dx, bi, bj, lds);
    else if (dx == 0) assemble_block<false, true>(v, p, ws, os, scale, dy, 0, bi, bj, lds);
    else assemble_block<false, false>(v, p, ws, os, scale, dy, dx, bi, bj, lds);
}

}  // namespace kfac
