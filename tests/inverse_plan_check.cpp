// Plays every launch of an inversion on the CPU, one number to a 128 x 128 block, from the schedule that the kernels use
// (inverse_plan.h).  The workgroups of a launch run in no order: nothing may be read that the same launch writes, nothing written
// twice, nothing read that was never written, and the result has to be the inverse.  Arguments: the smallest and the largest number
// of blocks.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1811_12019_amd/csrc/inverse_plan.h"

using namespace kfac;

namespace {

constexpr int NEVER = -2;
int faults = 0, launch = 0, blocks = 0;

void fault(const char* what) {
    if (++faults <= 20) printf("%d blocks, launch %d: %s\n", blocks, launch, what);
}

struct Cell {
    double value = 0;
    int written = NEVER;          // by which launch
    double read(const char* what) const {
        if (written == NEVER || written == launch) fault(what);
        return value;
    }
    void write(double v, const char* what) {
        if (written == launch) fault(what);
        value = v;
        written = launch;
    }
};

struct Matrix {
    int n;
    std::vector<double> S;
    std::vector<Cell> W, out, P, T, U;          // W, out: lower tiles; P: of even and odd steps; T, U: NBUF panels
    explicit Matrix(int n_) : n(n_), S(n * n), W(n * n), out(n * n), P(2), T(NBUF * n), U(NBUF * n) {
        srand(n);
        for (int i = 0; i < n; ++i)
            for (int j = 0; j <= i; ++j) S[i * n + j] = S[j * n + i] = (i == j ? 3.0 + 0.5 * n : 0.0) + rand() / (double)RAND_MAX - 0.5;
    }
    Cell& w(int I, int J) { return W[I * n + J]; }
    Cell& t(int step, int I) { return T[step % NBUF * n + I]; }
    Cell& u(int step, int I) { return U[step % NBUF * n + I]; }

    // the first step that a tile owes, and its old value
    int owed(int I, int J, int lo, int hi, double& old) {
        bool in_panel = false;
        const int first = owed_first(I, J, lo, hi, [&](int, int step, int slab) {
            in_panel = true;
            old = t(step, slab).read("old value in T");
        });
        if (!in_panel) old = w(I, J).read("old value");
        return first;
    }
    double products(int first, int last, int I, int J, double x) {
        for (int q = first; q <= last; ++q) x -= t(q, I).read("tile's T") * u(q, J).read("tile's U");
        return x;
    }
    void tile(int I, int J, const Group& g, bool single) {
        const int last = g.g0 + g.j;
        double old;
        int first = last;
        if (single) old = w(I, J).read("old value");
        else first = owed(I, J, g.g0, last, old);
        w(I, J).write(products(first, last, I, J, old), "tile");
    }
    void begin() {
        launch = -1;
        P[0].write(1 / S[0], "first pivot");
        w(0, 0).write(-1 / S[0], "first pivot's tile");
        for (int I = 1; I < n; ++I) {
            u(0, I).write(S[I * n], "first panel");
            for (int J = 1; J <= I; ++J) w(I, J).write(S[I * n + J], "working copy");
        }
    }
    void pivot(int k) {           // the look-ahead pivot: block k + 1; its slabs form T of the same rows
        const int c = k + 1;
        const double x = u(k, c).read("pivot's U");
        const double d = w(c, c).read("pivot's tile") - x * P[k & 1].read("P") * x;
        w(c, c).write(-1 / d, "pivot's tile");
        P[c & 1].write(1 / d, "next P");
        if (c == n - 1) out[c * n + c].write(1 / d, "last pivot's output");
    }
    void slab(int k, int I) {
        const int c = k + 1;
        const double p = P[k & 1].read("P");
        if (I == k) {             // block row k + 1 left of the diagonal, in block column k
            u(c, I).write(p * u(k, c).read("U of the pivot row"), "next panel");
            return;
        }
        const double own = u(k, I).read("U") * p;
        t(k, I).write(own, "T");
        if (I == c) return;
        auto product = [&](int q, int J) { return (q < k ? t(q, I).read("slab's T") : own) * u(q, J).read("slab's U"); };
        int first = chain_from(c);
        double x;
        if (I > c) {
            x = w(I, c).read("chain tile");
        } else if (I >= first) {
            first = I + 1;
            x = t(I, c).read("chain tile in T");
        } else {
            x = w(c, I).read("chain tile, turned");
        }
        if (k - first + 1 < 1 || k - first + 1 > GM + 1) fault("products of a half slab");
        for (int q = first; q <= k; ++q) x -= product(q, c);
        u(c, I).write(x, "next panel");
        if (I != k + 2) return;
        x = w(I, I).read("diagonal tile");
        for (int q = std::max(0, k - 1); q <= k; ++q) x -= product(q, I);
        w(I, I).write(x, "diagonal tile");
    }
    void stage(int s, bool out_owed) {
        launch = s;
        const Plan p = plan_of(n * NB, s);
        const int tiles = plan_workgroups(p, out_owed) - p.slabs;
        if (s < n - 1) {
            if (p.slabs != 2 * n) fault("half slabs");
            pivot(s);
            for (int I = 0; I < n; ++I) slab(s, I);
        } else {
            if (p.slabs != 2 * (n - 1)) fault("half slabs");
            for (int I = 0; I < n - 1; ++I) t(s, I).write(u(s, I).read("last U") * P[s & 1].read("last P"), "last T");
        }
        for (int e = 0; e < tiles; ++e) {
            int I, J;
            Group g;
            bool single;
            if (!stage_tile(p, n, s, e, I, J, g, single)) continue;
            if (J < 0 || J > I || I >= n || g.j >= GM) fault("no such tile");
            else tile(I, J, g, single);
        }
    }
    void outputs(bool out_owed) {
        launch = n;
        const int s = n - 1;
        for (int e = 0; e < n * (n + 1) / 2; ++e) {
            int I, J;
            tri_decode_blocked(n, e, I, J);
            if (J == s) continue;
            double x;
            if (I == s) {
                x = t(s, J).read("last T of the block row");
            } else {
                double old;
                int first = s;
                if (out_owed) first = owed(I, J, (s - 1) / GM * GM, s - 1, old);
                else old = w(I, J).read("old value");
                if (s - first > GM) fault("products of an output tile");
                x = products(first, s, I, J, old);
            }
            out[I * n + J].write(-x, "output");
        }
    }
    void check() {
        launch = n + 1;
        double worst = 0;
        for (int i = 0; i < n; i += std::max(1, n / 16))            // (some rows: S times the inverse is the unit matrix)
            for (int j = 0; j < n; ++j) {
                double x = 0;
                for (int q = 0; q < n; ++q) x += out[std::max(i, q) * n + std::min(i, q)].read("output that is not there") * S[q * n + j];
                worst = std::max(worst, std::fabs(x - (i == j)));
            }
        if (!(worst < 1e-9)) fault("the result is not the inverse");
    }
};

// Every matrix of a batch takes each of its stages once, in order, within the launches of the largest.
void check_schedule(int launches) {
    for (int n = 2; n <= launches; ++n)
        for (int i = 0; i < 6; ++i) {
            int taken = 0;
            for (int l = 0; l < launches; ++l) taken += takes_stage(n, launches, i, l);
            if (taken != n) fault("stages of a matrix in a batch");
        }
}

}  // namespace

int main(int argc, char** argv) {
    const int lo = argc > 1 ? atoi(argv[1]) : 2, hi = argc > 2 ? atoi(argv[2]) : 256;
    for (blocks = lo; blocks <= hi; ++blocks) {
        launch = -1;
        check_schedule(blocks);
        for (int out_owed = 0; out_owed < 2; ++out_owed) {
            Matrix m(blocks);
            m.begin();
            for (int s = 0; s < blocks; ++s) m.stage(s, out_owed);
            m.outputs(out_owed);
            m.check();
        }
    }
    printf("%d to %d blocks: %d faults\n", lo, hi, faults);
    return faults != 0;
}
