// CPU check of the search kernel's cut of a batch (split.h).
#include <cstdint>
#include <cstdio>

#include "split.h"

int main() {
    int failures = 0;
    const int64_t sizes[] = {1, 2, 63, 64, 65, 3'000, 20'000, 98'304, 200'000, 393'216, 1'000'000, 4'000'000, 64'000'000, INT32_MAX};
    for (int64_t n : sizes)
        for (int waves : {4, 8, 16})
            for (int per_cu : {1, 2, 3, 6, 16})
                for (int group : {1, 2, 4, 7, 8, 9, 16, 64}) {
                    const int cus = 256;
                    const samatch::SearchSplit s = samatch::search_split(n, cus, per_cu, waves, group);
                    const int64_t gmax = (int64_t)cus * per_cu, blocks = (s.chunks + s.group - 1) / s.group;
                    bool ok = s.per >= 1 && s.per <= 64 && s.chunks * s.per >= n && (s.chunks - 1) * s.per < n;
                    ok = ok && s.group >= 1 && s.group <= group && s.grid >= 1 && s.grid <= gmax;
                    // no workgroup has more chunks than an even share, in whole blocks, or one for each wave
                    const int64_t most = (blocks + s.grid - 1) / s.grid * s.group;
                    const int64_t share = (blocks + gmax - 1) / gmax * s.group;
                    ok = ok && (most <= share || most < waves + s.group);
                    if (!ok) {
                        std::printf("%lld reads, %d waves, %d workgroups per unit, group %d: %lld chunks of %d, group %d, grid %u\n",
                                    (long long)n, waves, per_cu, group, (long long)s.chunks, s.per, s.group, s.grid);
                        failures++;
                    }
                }
    std::printf("%s\n", failures ? "FAIL" : "ok");
    return failures ? 1 : 0;
}
