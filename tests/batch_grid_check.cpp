// Every launch of a batched search fits the 32-bit count of a launch's threads
// and reaches every work item, from one tile to the most a batch may hold.
#include <cstdio>
#include <initializer_list>

#include "kbmi_internal.h"

int main() {
    const int64_t most = 2147483647LL - 4096;
    for (int resident : {8, 2048, 4096})
        for (bool paced : {false, true})
            for (int64_t items : {int64_t(8), int64_t(8192), int64_t(67108856), int64_t(67108863),
                                  int64_t(67108864), int64_t(67108872), most}) {
                const kbmi::BatchGrid g = kbmi::batch_grid(items, resident, paced);
                const bool fits = g.grid >= 1 && (int64_t)g.grid * 64 < (int64_t(1) << 32);
                const bool all = (int64_t)g.grid * g.generations >= items &&
                                 (int64_t)g.grid * (g.generations - 1) < items;
                // Item numbers are 32-bit, the last generation's unused ones among them.
                const bool counted = (int64_t)g.grid * g.generations <= 2147483647LL;
                if (!fits || !all || !counted || (paced && g.grid != resident)) {
                    std::printf("%lld items, %d resident: %d workgroups, %d generations\n",
                                (long long)items, resident, g.grid, g.generations);
                    return 1;
                }
            }
    std::puts("batch grids ok");
    return 0;
}
