// The generic factor kernel's row ranges (factor_batch.h), counted on the CPU: a range is one chain of fp32 additions, so that it may have
// more than GENERIC_RANGE rows only where the launch has its 1,024 workgroups (rounded up to whole slabs); ranges cover the rows, none is empty.
#include <cstdio>

#include "../paper_1811_12019_amd/csrc/factor_batch.h"

using namespace kfac;

int main() {
    long faults = 0;
    for (int d : {1, 28, 64, 65, 129, 257, 513, 2049, 32768})
        for (long long R = 1; R <= 1000000000LL; R = R < 40000 ? R + 1 : R + R / 37) {
            Unfold u = {};
            u.d = d;
            u.R = (int)R;
            const FactorPlan p = plan_generic(u);
            const long long rows = p.rows_per_split, need = (R + 1023) / 1024 * p.ntiles;
            const long long most = need > GENERIC_RANGE ? need + GK : GENERIC_RANGE;
            faults += rows > most || rows % GK != 0 || (long long)p.nsplit * rows < R || (long long)(p.nsplit - 1) * rows >= R;
            faults += R <= 4 * GK && p.nsplit != 1;
        }
    printf("%ld faults\n", faults);
    return faults != 0;
}
