// The schedule of an inversion (inverse.hip): which launch forms, brings up to date and reads which block.  Integers only, host and
// device: tests/inverse_plan_check.cpp plays every launch of every block count on the CPU with one number to a block and looks for
// reads of what another workgroup of the same launch writes.
#pragma once

#include "common.h"

namespace kfac {

constexpr int NB = 128;          // elimination block = tile edge
static inline __host__ __device__ int nblk_of(int dim) { return (dim + NB - 1) / NB; }

// Steps are taken in groups of up to GM consecutive blocks, none of them the matrix's last.  Inside a group only what the chain
// needs is brought up to date; every other tile receives the group's rank-128 updates together, in one visit during the next
// group's launches, which cuts the traffic of the working copy by the group size.  The arithmetic per tile is the same sequence
// of fp32 operations as step-by-step updating.
constexpr int GM = 4;
struct Group {
    int g0;      // first step of a run of steps
    int m;       // its size (1 .. GM)
    int j;       // the last of them that a tile is to see, minus g0
};
// What the launch of a stage does for a matrix of n blocks (n >= 2).  Stage k <= n - 2 is step k, of the group [g0, g0 + GM):
//   * `slabs` half slabs (of pivot block k + 1's own only T).  Tile (I, k + 1) owes, in one visit, all steps from chain_from(k + 1) on.
//     The slabs of block k + 2 also bring their diagonal tile, which is kept up to date through step k - 2, up to step k.
//   * Diagonal tiles of the blocks the next pivots need are kept up to date one step behind, so that a look-ahead pivot never owes
//     more than one product: in a group's first launch blocks g0 + 3 .. g0 + 6 receive the whole group before, in the others
//     blocks k + 3 .. g0 + 6 step k - 1.
//   * The bulk: every other tile without an index inside the group receives the whole group before, in the group's launches but its
//     fourth (whose panel k + 1 takes the buffer of the first step of the group before).  The tiles of blocks g0 + 2 and g0 + 3
//     come first, in the group's first launch ("early" tiles): the panels k + 1 of the group's second and third launch read them.
//     (Block g0 + 1, whose panel the first launch forms, owes the group before and step g0: chain_from.)
// Stage n - 1: the panel of the last step, beside the tiles of all other blocks, which receive what the last group owes them, unless
// the output launch, which follows, is to do that (OUT_OWED).
struct Plan {
    Group g;             // the run of steps that the tiles see
    int slabs;           // workgroups of half slabs
    int d_begin, diag;   // diagonal tiles, from block d_begin on
    bool single;         // they see only the run's last step
    int g0, w;           // the group's first block and how many blocks it takes out of the bulk
    int early;           // number of early tiles of the group; early and lag tiles are one list, of which this launch takes
    int off, bulk;       // `bulk` tiles from `off` on
    int tiles;           // stage n - 1: all tiles but the last block's (left out where the output launch takes their updates)
};

static inline __host__ __device__ Plan plan_of(int dim, int stage) {
    const int n = nblk_of(dim);
    Plan p;
    p.d_begin = p.diag = p.g0 = p.w = p.early = p.off = p.bulk = p.tiles = 0;
    p.single = false;
    if (stage == n - 1) {
        p.slabs = 2 * (n - 1);
        p.tiles = n * (n - 1) / 2;
        p.g.g0 = (n - 2) / GM * GM;
        p.g.m = n - 1 - p.g.g0;
        p.g.j = p.g.m - 1;
        return p;
    }
    p.slabs = 2 * n;
    const int k = stage, g0 = k / GM * GM, j = k - g0, m = min(GM, n - 1 - g0);
    p.g0 = g0;
    p.w = min(GM, n - g0);
    if (j > 0) {
        p.g.g0 = g0;
        p.g.m = m;
        p.g.j = j - 1;
        p.single = true;
        p.d_begin = k + 3;
    } else {
        p.g.g0 = g0 - GM;
        p.g.m = GM;
        p.g.j = GM - 1;
        p.d_begin = g0 + 3;
    }
    if (k > 0) p.diag = max(0, min(g0 + 6, n - 1) - p.d_begin + 1);
    if (g0 > 0) {
        const int others = n - p.w, columns = max(0, p.w - 2);
        p.early = columns * others + (columns == 2);
        const int total = p.early + others * (others + 1) / 2, launches = min(m, GM - 1);
        const int first = launches == 1 ? total : max(p.early, (total + launches - 1) / launches);
        if (j == 0) {
            p.bulk = first;
        } else if (j < launches) {
            const int per = (total - first + launches - 2) / (launches - 1);
            p.off = first + (j - 1) * per;
            p.bulk = max(0, min(per, total - p.off));
        }
    }
    return p;
}
static inline int plan_workgroups(const Plan& p, bool out_owed) { return p.slabs + p.diag + p.bulk + (out_owed ? 0 : p.tiles); }
// The first step that the tiles of block column / row c owe when panel c is formed (by the launch of step c - 1): the working copy
// holds them through the step before it.
static inline __host__ __device__ int chain_from(int c) {
    const int r = c % GM;
    return max(0, r == 0 ? c - GM : r == 1 ? c - 1 - GM : c - r);
}
// index in the list of early and lag tiles -> (I, J): tiles of blocks g0 + 2 and g0 + 3, then the triangle over the blocks outside
// the group
__host__ __device__ __forceinline__ void bulk_decode(int n, int g0, int w, int early, int t, int& I, int& J) {
    const int others = n - w;
    if (t >= early) {
        tri_decode_blocked(others, t - early, I, J);
        if (I >= g0) I += w;
        if (J >= g0) J += w;
        return;
    }
    const int ci = t / others;
    if (ci >= w - 2) { I = g0 + 3; J = g0 + 2; return; }     // (the one tile of both)
    const int c = g0 + 2 + ci, o = t - ci * others, x = o < g0 ? o : o + w;
    I = max(c, x);
    J = min(c, x);
}

constexpr int NBUF = 2 * GM;     // panel buffers: buffer = step % NBUF

// Where a tile's old values come from: the working copy, or the T panel of the step that eliminated one of its blocks, as it lies
// (block column) or transposed (block row).
enum { OLD_W, OLD_T, OLD_T_TURNED };

// The first step that tile (I, J) owes of the steps lo .. hi.  Its old values are in the working copy, unless one of its blocks is among
// lo .. hi: such a tile was kept up to date until its later such block c was eliminated (when it became part of panel c: T_I (OLD_T) for a
// tile of block column c, T_J transposed (OLD_T_TURNED) for one of block row c, neither written to the working copy then), and owes
// the steps after c; old_in(kind, c, slab) is called with what that is.  The diagonal tile (c, c) is -P_c, which the pivot code did write.
template <class F>
__host__ __device__ __forceinline__ int owed_first(int I, int J, int lo, int hi, F&& old_in) {
    if (I >= lo && I <= hi) {                            // I is the later block (I >= J)
        if (I != J) old_in(OLD_T_TURNED, I, J);
        return I + 1;
    }
    if (J >= lo && J <= hi) {                            // I lies beyond
        old_in(OLD_T, J, I);
        return J + 1;
    }
    return lo;
}

// Tile `t` of those that a stage's launch takes beside its half slabs: (I, J) and the run of steps that it sees (single: its last
// only).  False: there is nothing to do for it.
__host__ __device__ __forceinline__ bool stage_tile(const Plan& p, int n, int stage, int t, int& I, int& J, Group& g, bool& single) {
    g = p.g;
    single = false;
    if (stage == n - 1) {
        tri_decode_blocked(n - 1, t, I, J);
        return !(I == J && I == n - 2);                  // (-P of the group's last step)
    }
    if (t < p.diag) {
        I = J = p.d_begin + t;
        single = p.single;
        return true;
    }
    bulk_decode(n, p.g0, p.w, p.early, p.off + t - p.diag, I, J);
    // -P of the group's last step; the diagonal tiles above
    if (I == J && (I == p.g0 - 1 || (I > p.g0 && I <= p.g0 + 6))) return false;
    g.g0 = p.g0 - GM;                                    // (the whole group before, whatever the diagonal tiles see)
    g.j = GM - 1;
    return true;
}

// Whether the matrix in place i of a batch, n blocks, takes its next stage in launch l of `launches`, as many as the largest matrix has
// blocks.  (A matrix's last stage touches all of its tiles: matrices with fewer blocks than the largest take it at different launches,
// none with the largest ones.)
static inline __host__ __device__ bool takes_stage(int n, int launches, int i, int l) {
    const int span = n == launches ? n : max(n, launches - 1 - i % 6);
    return l < span && (l + 1) * n / span > l * n / span;
}

}  // namespace kfac
