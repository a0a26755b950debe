// What the factor builders' launches share (factor.hip, factor_finish.hip): how a build is cut into tiles and row ranges, where its
// partial sums lie, and the argument block of a launch that serves many builds.
#pragma once

#include "factor_tile.h"
#include "factor_repack.h"
#include "factor_shared.h"

namespace kfac {

struct FactorPlan {
    int tw;          // tile width (matrix-core builds)
    int tiles_dim;   // tiles per dimension
    int ntiles;      // lower-triangular tiles
    int nsplit;
    int rows_per_split;
    int tile_floats; // partial sums of a tile of one split (matrix-core builds)
    size_t ws_bytes;
};

// Tile width and row split of a matrix-core build.  `share`: how the builds of a call are cut (rows_of, takes_wide): the rows of a
// workgroup, plus SHARE_WIDE if matrices of more than 128 columns get 256-wide tiles, plus SHARE_PLANES if the tensor is read as
// planes (the address decides that, once, on the host: worked out by the kernels it cost each launch 0.2 to 0.5 us).  A matrix of up to
// 128 (64) columns is one tile of that width.
constexpr int SHARE_WIDE = 1 << 20, SHARE_PLANES = 1 << 21;
constexpr int SHARE_TURN_SHIFT = 24;         // (for the tile kernel: the build's `turn`, see unit_of)
constexpr int ROWS_PER_WG_MAX = 6400, ROWS_PER_WG_MAX_F32 = 1600;
constexpr int ROWS_PER_WG_MIN = 512, ROWS_PER_WG_MIN_F32 = 64;
constexpr int SHARE_LEAST = 1024, SHARE_LEAST_WIDE = 1600, SHARE_LEAST_F32 = 128;    // the fewest rows rows_of gives a workgroup (256-wide)

// splits that keep a build's partial sums below 34 MB (256-wide tiles: 67 MB), unless a workgroup's rows would pass the maximum
static inline __host__ __device__ int most_splits(int R, int tw, int ntiles, bool f32) {
    const int cap = (tw == 256 ? 256 : 512) / ntiles, need = ceil_div(R, f32 ? ROWS_PER_WG_MAX_F32 : ROWS_PER_WG_MAX);
    const int most = R / (f32 ? ROWS_PER_WG_MIN_F32 : ROWS_PER_WG_MIN);
    const int ns = cap > need ? cap : need;
    return ns > most ? (most > 1 ? most : 1) : (ns > 1 ? ns : 1);
}

// multiples of 8 keep a row range on one XCD
static inline __host__ __device__ int xcd_splits(int ns) { return ns >= 8 ? ns / 8 * 8 : ns; }

// The same for a layer whose tap pairs share their sums.
constexpr int SHARED_ROWS_LEAST = 400, SHARED_ROWS_LEAST_F32 = 80;
static inline __host__ __device__ SharedPlan plan_shared(const View& v, int share) {
    SharedPlan p;
    const Unfold& u = v.u;
    const bool f32 = u.dtype == KFAC_F32;
    p.tw = u.C <= 64 ? 64 : u.C <= 128 || f32 || !(share & SHARE_WIDE) ? 128 : 256;
    p.T = ceil_div(u.C, p.tw);
    p.ntl = p.T * (p.T + 1) / 2;
    p.nf = p.T * p.T;
    p.per[0] = p.ntl + 12 * p.nf;
    p.per[1] = p.per[2] = 2 * p.ntl + 4 * p.nf;
    p.per[3] = 4 * p.ntl;
    // Three quarters of a dense tile's rows: an entry's sum is then no longer a chain of fp32 additions than there (with as many rows
    // the error against 64 bits was up to 1.6 times the dense form's, now it is nowhere larger).
    const int share_rows = (share & (SHARE_WIDE - 1)) * 3 / 4;
    const int rows = u.N * (u.H - 1) * (u.W - 1);
    const int memory = (p.tw == 256 ? 256 : 512) / p.per[0], need = ceil_div(rows, f32 ? ROWS_PER_WG_MAX_F32 : ROWS_PER_WG_MAX);   // (most_splits)
    const int cap = memory > need ? memory : need;
    const int least = rows / (f32 ? SHARED_ROWS_LEAST_F32 : p.per[0] > 128 ? 640 : SHARED_ROWS_LEAST);   // (512 channels, 1,152 rows: not two)
    int ns = ceil_div(rows, share_rows);
    if (ns > cap) ns = cap;
    if (ns > least) ns = least > 1 ? least : 1;
    p.ns[0] = xcd_splits(ns);
    // (written out: as a loop over the classes the plan stays an array in scratch memory, which every workgroup waits for)
    auto strips = [&](int rows_of_class) { const int n = ceil_div(rows_of_class, share_rows); return n < p.ns[0] ? n : p.ns[0]; };
    p.ns[1] = strips(u.N * (u.W - 1));
    p.ns[2] = strips(u.N * (u.H - 1));
    p.ns[3] = strips(u.N);
    p.first[0] = 0;
    p.first[1] = p.ns[0] * p.per[0];
    p.first[2] = p.first[1] + p.ns[1] * p.per[1];
    p.first[3] = p.first[2] + p.ns[2] * p.per[2];
    p.first[4] = p.first[3] + p.ns[3] * p.per[3];
    p.rows = ceil_div(rows, p.ns[0]);
    p.ws_bytes = ((size_t)p.first[4] * p.tw * p.tw + (size_t)9 * p.ns[0] * p.T * p.tw) * sizeof(float);
    return p;
}

static inline __host__ __device__ FactorPlan plan_tiles(const View& v, int share) {
    FactorPlan p;
    const int D = v.u.d, R = v.u.R;
    const bool f32 = v.u.dtype == KFAC_F32;
    p.tw = D <= 64 ? 64 : D <= 128 || f32 || !(share & SHARE_WIDE) ? 128 : 256;
    p.tiles_dim = ceil_div(D, p.tw);
    p.ntiles = p.tiles_dim * (p.tiles_dim + 1) / 2;
    const int most = most_splits(R, p.tw, p.ntiles, f32);
    int ns = ceil_div(R, share & (SHARE_WIDE - 1));
    if (ns > most) ns = most;
    ns = xcd_splits(ns);
    p.rows_per_split = ceil_div(ceil_div(R, ns), 64) * 64;
    p.nsplit = ceil_div(R, p.rows_per_split);
    p.tile_floats = tile_floats(p.tw, p.ntiles);
    p.ws_bytes = p.nsplit > 1 ? (size_t)p.nsplit * ((size_t)p.ntiles * p.tile_floats + (size_t)p.tiles_dim * p.tw) * sizeof(float) : 0;
    return p;
}

// The generic kernel's builds (factor.hip).
constexpr int GT = 64;   // output tile edge
constexpr int GK = 16;   // unfolded rows per LDS stage
// Row ranges: at most 160, since the second pass reads them all (12,544 rows of 28 columns with 392 29.2 us, with 160 23.1, with 96 26.7), but
// as many as keep a range, which is one chain of fp32 additions, at 128 rows or below.  Channels-last tensors off the 16-byte grid, bf16, 64
// columns, with 160 ranges and so: 50,176 rows 50 us, error against 64 bits 5.3e-7, and 44, 1.9e-7; 401,408 301, 3.9e-6, and 127, 8.1e-7.
constexpr int GENERIC_SPLITS = 160, GENERIC_RANGE = 128;
static inline __host__ __device__ FactorPlan plan_generic(const Unfold& u) {
    FactorPlan p;
    p.tiles_dim = ceil_div(u.d, GT);
    p.ntiles = p.tiles_dim * (p.tiles_dim + 1) / 2;
    int want = ceil_div(1024, p.ntiles);                       // (four workgroups to a CU)
    // Two slabs to a workgroup, whose time is the latency of its few trips to memory (512 rows of 145 columns: four slabs 11.8 us, two
    // 8.1, one 6.1 and 0.8 more for the second pass); up to 64 rows stay in one, without that pass.
    const int most = ceil_div(u.R, GENERIC_RANGE) > GENERIC_SPLITS ? ceil_div(u.R, GENERIC_RANGE) : GENERIC_SPLITS;
    const int slabs = ceil_div(u.R, 2 * GK), max_split = u.R <= 4 * GK ? 1 : slabs < most ? slabs : most;
    p.nsplit = want < 1 ? 1 : (want > max_split ? max_split : want);
    if (p.nsplit < 1) p.nsplit = 1;
    p.rows_per_split = ceil_div(ceil_div(u.R, p.nsplit), GK) * GK;
    p.nsplit = ceil_div(u.R, p.rows_per_split);
    p.ws_bytes = p.nsplit > 1 ? (size_t)p.nsplit * p.ntiles * GT * GT * sizeof(float) : 0;
    return p;
}

// The workspace of a matrix-core build: the repacked tensor, if there is one, then the partial sums.
static inline __host__ __device__ Partial partial_of(const View& v, const FactorPlan& p, void* ws) {
    Partial q;
    q.tiles = (gfloat*)(ws ? (unsigned char*)ws + repack_bytes(v) : nullptr);
    q.sums = q.tiles + (size_t)p.nsplit * p.ntiles * p.tile_floats;
    return q;
}

static inline __device__ gfloat* shared_ws(const View& v, void* ws) { return (gfloat*)((unsigned char*)ws + repack_bytes(v)); }

// Where an item's result goes.
static __host__ __device__ __forceinline__ OutSpec out_spec(const kfac_factor_item& it) {
    OutSpec o;
    o.decay = it.decay;
    o.one_minus = 1.0f - it.decay;
    if (it.running) { o.dst = (gfloat*)it.running; o.mode = OUT_EMA; }
    else { o.dst = (gfloat*)it.out; o.mode = it.packed ? OUT_PACKED : OUT_PLAIN; }
    return o;
}

// ---- batched launches: many factor builds in one grid -------------------------------------------------------------
constexpr int FMAXB = 120;

struct FBatch {
    const kfac_factor_item* table;   // device table, or nullptr -> `single`
    kfac_factor_item single;
    int count;
    int index[FMAXB];                // table index of the i-th build of this launch
    int share[FMAXB];                // plan_tiles' argument for it
    int prefix[FMAXB + 1];           // workgroup prefix sums
};

__device__ __forceinline__ int fbatch_locate(const FBatch& b, int wg, int& local) {
    int lo = 0, hi = b.count;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (b.prefix[mid] <= wg) lo = mid; else hi = mid;
    }
    local = wg - b.prefix[lo];
    return lo;
}

// (a launch of builds that are not read as planes: PLANES = false)
template <bool PLANES = true>
__device__ __forceinline__ void fbatch_item(const FBatch& b, int m, kfac_factor_item& it, Unfold& u, View& v) {
    if (b.table) it = uniform(b.table[b.index[m]]);
    else it = b.single;
    if (it.op == KFAC_OP_FACTOR_A) make_unfold_A(&it.desc, &u); else make_unfold_G(&it.desc, &u);
    make_view(u, &v);
    if (PLANES && (b.share[m] & SHARE_PLANES)) planes_view(u, &v);
}

// Tiles of the builds of `b`; KIND 0: bf16, 1: fp16, 2: fp32 (factor_launch.h).
template <int KIND>
int launch_tiles(int tw, bool planes, const FBatch& b, hipStream_t stream);

// Second passes of the builds of `b` (factor_finish.hip): builds of few row ranges or shared sums, of many ranges, of shared sums in
// (channel, tap) order.
enum { FINISH_FEW, FINISH_MANY, FINISH_CHANNELS, FINISH_LISTS };
int launch_factor_finish(const FBatch& b, int list, hipStream_t stream);

// Workgroups of the second pass of split rows.
constexpr int MANY_SPLITS = 32;
static inline __host__ __device__ int reduce_wgs(const View& v, const FactorPlan& p) {
    return p.ntiles * (p.tw / 32) * (p.tw / 32) * (p.nsplit >= MANY_SPLITS ? 4 : 1) + (v.u.has_bias ? ceil_div(v.u.d, 256) : 0);
}

}  // namespace kfac
