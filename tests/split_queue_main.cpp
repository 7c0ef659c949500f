// Drives the slot arithmetic of the split streams' queue (csrc/split.hpp) as
// the waves do, one reservation after another (compiled by
// tests/test_split_queue.py).  argv: slots, batches, tasks each batch asks
// for, and what was asked for before.  No slot may be given out twice, none
// beyond the queue; every slot that the task kernels visit is written (a task
// or the mark for none); a batch that gets no slots streams by itself.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "split.hpp"

int main(int argc, char** argv) {
    if (argc != 5) return 2;
    const uint32_t cap = (uint32_t)strtoul(argv[1], nullptr, 10);
    const uint64_t batches = strtoull(argv[2], nullptr, 10);
    const uint32_t want = (uint32_t)strtoul(argv[3], nullptr, 10);
    gd::SplitCount asked = (gd::SplitCount)strtoull(argv[4], nullptr, 10);
    const bool fresh = asked == 0;
    std::vector<char> written(cap, 0);
    uint64_t given = 0, alone = 0;
    for (uint64_t b = 0; b < batches; ++b) {
        const gd::SplitCount before = asked;
        asked += want;  // the wave's atomic addition
        if (gd::split_fits(before, want, cap)) {
            for (uint32_t i = 0; i < want; ++i) {
                if (before + i >= cap || written[before + i]) {
                    printf("slot %llu given twice or beyond the queue in batch %llu\n",
                           (unsigned long long)(before + i), (unsigned long long)b);
                    return 1;
                }
                written[before + i] = 1;
            }
            given += want;
        } else {
            for (gd::SplitCount at = before; at < cap; ++at) written[at] = 1;  // marked as none
            ++alone;
        }
    }
    const uint32_t used = gd::split_used(asked, cap);
    for (uint32_t i = 0; fresh && i < used; ++i)
        if (!written[i]) {
            printf("slot %u is visited but was never written\n", i);
            return 1;
        }
    if (!fresh && given) {
        printf("%llu tasks given out of a full queue\n", (unsigned long long)given);
        return 1;
    }
    printf("given %llu alone %llu used %u\n", (unsigned long long)given, (unsigned long long)alone, used);
    return 0;
}
