// How the factor builds of a call are cut, on the host: which kernel serves a build, rows of a workgroup and width of its tiles, and the
// scratch that covers every call a build may be part of.
#pragma once

#include <algorithm>

#include "factor_batch.h"

namespace kfac {

static bool item_unfold(const kfac_factor_item& it, Unfold* u) {
    if (it.op == KFAC_OP_FACTOR_A) return make_unfold_A(&it.desc, u);
    if (it.op == KFAC_OP_FACTOR_G) return make_unfold_G(&it.desc, u);
    return false;
}

// Whether the matrix-core kernels take a build whose tensor lies at x.
static bool tile_eligible(const Unfold& u, const void* x, View* v) {
    if (!make_view(u, v)) return false;
    if (reads_planes(u, x)) planes_view(u, v);
    return ((uintptr_t)x & (v->repack ? (u.dtype == KFAC_F32 ? 3 : 1) : 15)) == 0;
}

// How a build is served.
enum Route { ROUTE_TILE, ROUTE_GENERIC };

// A build that would have to be repacked first is left to the generic kernel while it is so small that the launch this saves weighs more
// than the arithmetic (bf16, 512 rows of 145 columns: 10.9 us, and 20.9 repacked; 256 of 289 11.0 and 20.9), unless many builds share the
// repacking and tile launches.  A single build would be the faster for it up to four times that size (512 of 289 12.6 and 26.8), but not
// a call of several, whose builds are cut as they would be alone (six of them 30.4 and 27.9; six of 98 rows of 1,025 columns 57.6 and
// 25.6).  Of many rows the second pass reads too many sums (49,000 rows of 6 columns 60.7 us, as a tile 20.4;
// 12,544 rows of 28 columns of a 3x3 layer 23.1 and 30.2).
constexpr long long GENERIC_MACS = 1 << 25;
constexpr int GENERIC_ROWS = 16384;

// Planes read as they lie save the repacking, but not the second launch: small builds of few rows stay there too (bf16, 2,048 rows of 63
// columns 14.3 us, 1,024 of 145 12.1).  From 4,096 rows on the tile is the faster one (8,192 rows of 63 columns 14.1 us).
constexpr int GENERIC_PLANE_ROWS = 4096;

static Route route_of(const Unfold& u, const void* x, bool many, View* v) {
    if (!tile_eligible(u, x, v)) return ROUTE_GENERIC;
    const int rows = v->repack ? GENERIC_ROWS : v->planes ? GENERIC_PLANE_ROWS : 0;
    return !many && u.R < rows && (long long)u.R * u.d * u.d <= GENERIC_MACS ? ROUTE_GENERIC : ROUTE_TILE;
}

// The work of a call's builds of one element size, in rows of 128 x 128 tiles, cut into 128- and into 256-wide tiles; of the
// builds that would be cut into 256-wide ones, in 128-wide tiles, and in rows and workgroups of 256-wide ones (add_wide_work).
struct TileWork {
    double narrow = 0, wide = 0, over = 0, wide_rows = 0;
    double area = 0, filled = 0;                                 // their columns, padded to multiples of 256 and not, squared, times rows
    int wide_wgs = 0;
};
static void add_work(TileWork& w, const View& v) {
    const double cols = v.shared ? v.u.C : v.u.d, padded = 256.0 * ceil_div((int)cols, 256);
    if (cols > 128) {
        w.area += padded * padded * v.u.R;
        w.filled += cols * cols * v.u.R;
    }
    if (v.shared) {
        const double n = ceil_div(v.u.C, 128), m = ceil_div(v.u.C, 256), tiles = v.u.C <= 64 ? 13 * 0.5 : 0.5 * n * (n + 1) + 12 * n * n;
        w.narrow += tiles * v.u.R;
        w.wide += (v.u.C <= 128 ? tiles : 2.0 * m * (m + 1) + 48 * m * m) * v.u.R;
        if (v.u.C > 128) w.over += tiles * v.u.R;
        return;
    }
    const double n = ceil_div(v.u.d, 128), m = ceil_div(v.u.d, 256), tiles = 0.5 * n * (n + 1);
    w.narrow += tiles * v.u.R;
    w.wide += (v.u.d <= 128 ? tiles : 2.0 * m * (m + 1)) * v.u.R;
    if (v.u.d > 128) w.over += tiles * v.u.R;
}

// How they are cut (in a call of few builds each by its own work: CallCut).  The rows of a workgroup: half of what
// each of the 768 workgroups that run at a time would get of all the work, within limits.  More leaves the chip waiting for the
// last ones (18,816 rows of the first stage's layers at 3200 to a workgroup 119 us, at 6400 181 us), less adds partial sums, each
// as much traffic as a finished tile, for nothing (the third stage's 18 layers at 1568 rows: 151 us unsplit, 334 us in two).  When
// there is little work the launch of the second pass weighs too.
// (768: three workgroups to a CU, as 16-bit tiles run.  Of fp32 ones two do, and the line is from when it was three: of 239 fp32 calls,
// counted in 512, most take the same time within 3 % and calls of little work less, layers 12 to 30 of ResNet-50 at batch 2 198 us instead of
// 250, all at batch 1 466 and 495; but chains of additions, and the errors, would be up to half as long again.)
static int rows_of(const TileWork& w, bool f32) {
    const double per_slot = w.narrow / 768;
    const double least = f32 ? (per_slot < 100 ? SHARE_LEAST_F32 : 256) : (per_slot < 512 ? SHARE_LEAST : SHARE_LEAST_WIDE);
    return (int)std::min(std::max(0.52 * per_slot, least), (double)(f32 ? ROWS_PER_WG_MAX_F32 : ROWS_PER_WG_MAX));
}

static void add_wide_work(TileWork& w, const View& v, int rows) {
    if (v.shared) {
        if (v.u.C <= 128) return;
        const SharedPlan p = plan_shared(v, rows | SHARE_WIDE);
        w.wide_rows += (double)p.per[0] * v.u.R;
        w.wide_wgs += p.first[4];
    } else if (v.u.d > 128) {
        const FactorPlan p = plan_tiles(v, rows | SHARE_WIDE);
        w.wide_rows += (double)p.ntiles * v.u.R;
        w.wide_wgs += p.ntiles * p.nsplit;
    }
}

// Width (16-bit inputs): a 256-wide tile halves the operand traffic per product, but a workgroup fills a CU, its epilogue overlaps with
// nothing and a matrix is padded to multiples of 256.  It is the better one for workgroups enough to give most CUs one, of rows enough to
// outweigh the epilogue, with little padding, and if most of the call's work is in matrices of more than 128 columns, or much is.  The rows
// of a range, and so the error, are those of 128-wide tiles.  Runs of ResNet-50's layers in bf16, 128- and 256-wide, us:
//     all 54, batch 12 562 and 570, 18 719 and 676, 24 926 and 819, 32 1117 and 960      (workgroups of 1,444, 2,072, 2,785, 3,265 rows)
//     layers 23 to 43, batch 8 169 and 199, 16 285 and 277, 32 408 and 368, 64 725 and 545            (1,046, 1,408, 2,817, 5,021 rows)
//     layers 43 to 53, batch 16 227 and 257, 32 297 and 295, 64 404 and 353                                  (766, 1,254, 2,508 rows)
//     one 1x1 layer of 256 columns (a third more work in 256-wide tiles, but full ones) at 56 x 56, batch 64 114 and 108, 256 351 and 310
//     the first convolution (224 of 256 columns; narrow), batch 64 111 and 120, 256 374 and 413                   (256 and 492 workgroups)
//     one 3x3 layer of 256 channels at 14 x 14, batch 32 33 and 37, 256 115 and 99, 512 193 and 159             (77, 272, 272 workgroups)
//     the first 12 (0.48 of the work in wide matrices), batch 32 302 and 317, 64 544 and 563, 128 1103 and 981 (1.1, 2.2, 4.4 M tile rows)
// One matrix, near the lines (workgroups of rows on average): 132 of 1,853 60 and 66, 144 of 1,568 46 and 49, 160 of 1,960 76 and 59, 181 of
// 1,663 61 and 56, 180 of 1,436 60 and 62, 236 of 1,209 64 and 61, 225 of 1,666 95 and 72: there the line in rows leaves up to a quarter;
// just more workgroups than CUs, 270 of 6,272, 272 and 288.  Runs with 0.4 to 0.6 of the work in wide matrices, by tile rows: 1.1 M 281 and
// 301, 1.4 324 and 293, 1.7 386 and 368, 2.0 447 and 456, 2.2 488 and 518, 2.7 587 and 531, 2.8 658 and 590, 3.3 785 and 779.  A call of few
// builds that take both widths has two launches: layers 7 to 13 at batch 55 291 us, all narrow 273.
// Against the lines before it (24,000 rows of 128-wide tiles to one of 768 slots, padding below 15 %) 63 of 204 runs of 1 to 54 layers,
// 5 to 512 images and both layouts are faster by 2 to 94 %, the others within the spread of repeated runs.  (Always 6,400 rows to a 256-wide
// workgroup fill fewer CUs and add up longer chains.)
constexpr int WIDE_WGS = 150, WIDE_ROWS = 1900;
constexpr double WIDE_PADDING = 1.25, WIDE_PADDING_FULL = 1.34, WIDE_PART = 0.7, WIDE_MUCH = 2.5e6, WIDE_ALWAYS = 100000 * 768.0;
static bool takes_wide(const TileWork& w, int rows) {
    if (w.narrow >= WIDE_ALWAYS) return true;                    // so much that padding and the launch's end do not show
    return rows >= SHARE_LEAST_WIDE && w.wide_wgs >= WIDE_WGS && w.wide_rows >= (double)WIDE_ROWS * w.wide_wgs &&
           (w.wide <= WIDE_PADDING * w.narrow || (w.wide <= WIDE_PADDING_FULL * w.narrow && w.area <= WIDE_PADDING * w.filled)) &&
           (w.over >= WIDE_PART * w.narrow || w.wide_rows >= WIDE_MUCH);
}

// The scratch of a matrix-core build, for every call it may be part of: the work of a call is at least the build's own, a workgroup's rows grow
// with it (rows_of), and the fewer rows, the more partial sums.  (The factors of ResNet-50 from channels-last bf16 tensors: 1.90 GB at batch
// 32, 3.16 GB at batch 128; with the fewest rows of any call 1.93 and 3.17; fp32 at 32 2.28 and 2.44.)
static size_t tiles_ws_bytes(const View& v) {
    TileWork own;
    add_work(own, v);
    const bool f32 = v.u.dtype == KFAC_F32;
    const int rows = rows_of(own, f32), wide = std::max(rows, SHARE_LEAST_WIDE) | SHARE_WIDE;       // (see takes_wide)
    if (v.shared) return std::max(plan_shared(v, rows).ws_bytes, f32 ? 0 : plan_shared(v, wide).ws_bytes);
    return std::max(plan_tiles(v, rows).ws_bytes, f32 ? 0 : plan_tiles(v, wide).ws_bytes);
}

static size_t item_ws_bytes(const Unfold& u) {
    size_t need = plan_generic(u).ws_bytes;                    // any kernel may serve the build
    View v;
    if (make_view(u, &v)) {                                    // (with the place of a repacked copy: the address decides whether there is one)
        need = std::max(need, repack_bytes(v) + tiles_ws_bytes(v));
    }
    return align_up(need, 256);
}

// How a call is cut.
struct CallCut {
    bool many;                   // by the work of all its builds (of one element size), else each build by its own
    int share16, share32;
    // Few builds: each is cut as it would be in a call of its own, so that its result is the same to the last bit (kfac.h).  By
    // the work of the whole call, one to seven layers of ResNet-50 at batch 2 to 32 take between 26 % less time (five layers of the
    // third stage at batch 8: 52 instead of 70 us) and 11 % more (four layers around the second stage's start at batch 8: 70 instead
    // of 63 us).
    int share(const View& v) const {
        const bool f32 = v.u.dtype == KFAC_F32;
        const int flag = v.planes ? SHARE_PLANES : 0;
        if (many) return (f32 ? share32 : share16) | flag;
        TileWork own;
        add_work(own, v);
        const int rows = rows_of(own, f32);
        if (f32) return rows | flag;
        add_wide_work(own, v, rows);
        return rows | flag | (takes_wide(own, rows) ? SHARE_WIDE : 0);
    }
};
static CallCut cut_call(const kfac_factor_item* host, int count) {
    CallCut cut = {false, 0, 0};
    Unfold u;
    View v;
    int n_tile = 0;
    for (int i = 0; i < count; ++i) n_tile += item_unfold(host[i], &u) && route_of(u, host[i].x, true, &v) == ROUTE_TILE;
    cut.many = n_tile >= 16;
    if (!cut.many) return cut;
    TileWork work16, work32;
    for (int pass = 0; pass < 2; ++pass) {
        for (int i = 0; i < count; ++i) {
            item_unfold(host[i], &u);
            if (route_of(u, host[i].x, true, &v) != ROUTE_TILE || (pass && u.dtype == KFAC_F32)) continue;
            if (pass) add_wide_work(work16, v, cut.share16);
            else add_work(u.dtype == KFAC_F32 ? work32 : work16, v);
        }
        cut.share16 = rows_of(work16, false);
    }
    cut.share32 = rows_of(work32, true);
    if (takes_wide(work16, cut.share16)) cut.share16 |= SHARE_WIDE;
    return cut;
}

}  // namespace kfac
