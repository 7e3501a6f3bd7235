// CPU check of the work items of the kernels that take groups in a fixed order (group_items.h): for
// every launch every (group, part) is taken once, and the XCDs get about equal numbers of blocks with
// work.  Prints "kernel groups n_group|parts|items taken once|all items|busiest XCD / mean".
#include <algorithm>
#include <cstdio>
#include <vector>

#include "group_items.h"

using namespace fdx;

static void check(const char *name, size_t groups, int n_group, const GroupItems &o,
                  uint32_t per_block) {
    std::vector<uint32_t> taken(groups * o.parts);
    size_t busy[8] = {}, blocks = 0, out = 0;
    for (uint32_t vb = 0; vb < o.blocks; vb++) {
        const size_t b = xcd_run_block(vb, o.run);
        bool work = false;
        for (uint32_t w = 0; w < per_block; w++) {
            const size_t item = b * per_block + w;            // part x groups + group
            if (item / groups >= o.parts) continue;
            taken[item]++;
            work = true;
        }
        busy[vb % 8] += work;
        blocks += work;
    }
    for (uint32_t t : taken) out += t == 1;
    std::printf("%s %zu %d|%u|%zu|%zu|%.3f\n", name, groups, n_group, o.parts, out, taken.size(),
                8.0 * *std::max_element(busy, busy + 8) / blocks);
}

int main() {
    for (size_t groups : {1ul, 2ul, 7ul, 33ul, 130ul, 511ul, 512ul, 1000ul, 4097ul, 16383ul, 16384ul,
                          16385ul, 70001ul, 300000ul})
        for (int n_group : {1, 8, 16, 17, 64, 80, 81, 100, 128, 256, 512}) {
            check("density", groups, n_group, density_items(groups, n_group), 4);
            check("cut", groups, n_group, cut_items(groups, n_group), 1);
        }
    return 0;
}
