// How the factor builds' work lists are dealt to the XCDs (factor_tile.h), counted on the CPU: every unit goes to exactly one workgroup of
// the padded grid, no two XCDs' shares of a launch of builds differ by more than one unit, and an XCD's share of a build is contiguous.
#include <cstdio>
#include <vector>

#include "../paper_1811_12019_amd/csrc/factor_tile.h"

using namespace kfac;

int main() {
    int faults = 0;
    for (int first = 0; first < 8; ++first) {
        int turn = first, load[8] = {}, total = 0;
        for (int work = 0; work <= 300; ++work) {
            std::vector<int> seen(work, 0);
            int last[8];
            for (int& l : last) l = -1;
            for (int wg = 0; wg < (work + 7) / 8 * 8; ++wg) {
                const int unit = unit_of(work, wg, turn), xcd = wg & 7;
                if (unit < 0) continue;
                if (unit >= work || seen[unit]++) { ++faults; continue; }
                if (last[xcd] >= 0 && unit != last[xcd] + 1) ++faults;
                last[xcd] = unit;
                ++load[xcd];
                ++total;
            }
            for (int s : seen) faults += s != 1;
            for (int l : load) faults += l < total / 8 || l > (total + 7) / 8;
            turn = next_turn(turn, work);
        }
    }
    printf("%d faults\n", faults);
    return faults != 0;
}
