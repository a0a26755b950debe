// The scratch of the factor builds (factor_cut.h), counted on the CPU: random calls of 1 to 120 builds of any shape, type, layout and address.
// However a call cuts its builds, each one's partial sums and repacked copy fit what kfac_factor_workspace_bytes asks for it.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "../paper_1811_12019_amd/csrc/factor_cut.h"

using namespace kfac;

int main() {
    std::mt19937 rng(1);
    auto below = [&](int n) { return (int)(rng() % n); };
    auto log_uniform = [&](double lo, double hi) { return (int)(lo * std::pow(hi / lo, rng() / 4294967296.0)); };
    long faults = 0, tiles = 0, wide = 0, shared = 0, generic = 0, several = 0;
    for (int call = 0; call < 30000; ++call) {
        std::vector<kfac_factor_item> items;
        const int n = below(2) ? log_uniform(1, 121) : log_uniform(1, 8), dtype = below(4), largest = log_uniform(8, 300);
        while ((int)items.size() < n) {
            kfac_factor_item it = {};
            const int k = below(2) ? 1 : below(3) ? 3 : 7, hw = log_uniform(1, 115);
            it.desc = {log_uniform(1, largest), log_uniform(1, 2200), hw, below(3) ? hw : log_uniform(1, 60), log_uniform(1, 2200), k, k,
                       below(3) ? 1 : 2, below(4) ? k / 2 : 0, below(2), below(2), dtype < 3 ? dtype : below(3), below(2)};
            it.op = below(2);
            it.x = (const void*)(size_t)(1 << 20 | (below(4) ? 0 : 2 * below(8)));
            Unfold u;
            if (!item_unfold(it, &u)) continue;
            items.push_back(it);
        }
        const CallCut cut = cut_call(items.data(), n);
        for (const kfac_factor_item& it : items) {
            Unfold u;
            View v;
            item_unfold(it, &u);
            size_t need;
            if (route_of(u, it.x, cut.many, &v) != ROUTE_TILE) {
                need = plan_generic(u).ws_bytes;
                ++generic;
            } else {
                const int share = cut.share(v);
                const FactorPlan p = v.shared ? FactorPlan() : plan_tiles(v, share);
                const SharedPlan q = v.shared ? plan_shared(v, share) : SharedPlan();
                need = repack_bytes(v) + (v.shared ? q.ws_bytes : p.ws_bytes);
                ++tiles;
                shared += v.shared;
                wide += (v.shared ? q.tw : p.tw) == 256;
                several += !v.shared && p.nsplit > 1;
            }
            faults += need > item_ws_bytes(u);
        }
    }
    printf("%ld faults\n", faults + (wide < 1000) + (shared < 1000) + (generic < 1000) + (several < 1000));
    fprintf(stderr, "%ld tiles (%ld wide, %ld shared, %ld split), %ld generic\n", tiles, wide, shared, several, generic);
    return faults != 0;
}
