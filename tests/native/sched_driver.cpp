// Schedule positions of the matrix-core attention kernels.  Reads lines "W cus total s_0 ... s_total-1" (work of the units, by
// decreasing length) and prints the order and, round after round, the unit each of the W workgroups takes by position.
#include <cstdio>
#include <vector>

#include "../../paper_2503_05096_amd/csrc/adaspec_internal.h"

int main()
{
    int W, cus, total;
    while (scanf("%d %d %d", &W, &cus, &total) == 3) {
        std::vector<int> work(total);
        for (int &w : work)
            if (scanf("%d", &w) != 1) return 1;
        int size[adaspec::kSchedSamples] = {};
        if (adaspec::sched_asks_sizes(total, W, cus))
            for (int k = 0; k < adaspec::kSchedSamples; ++k) size[k] = work.at(adaspec::sched_sample(k, total, W, cus));
        const int order = adaspec::sched_order(total, W, cus, adaspec::kEvenRounds, size);
        printf("%d", order);
        for (int r = 0; r * W < total; ++r)
            for (int w = 0; w < W; ++w) printf(" %d", adaspec::sched_position(r, w, W, cus, order));
        printf("\n");
    }
    return 0;
}
