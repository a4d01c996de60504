// How a batch in input order is cut for the search kernel.  Plain C++ so that
// a CPU test can check it over the whole range of sizes and settings.
#pragma once

#include <algorithm>
#include <cstdint>

namespace samatch {

struct SearchSplit {
    int per;         // reads of a chunk, at most 64
    int64_t chunks;
    int group;       // chunks of a block, which one workgroup takes
    unsigned grid;   // workgroups
};

// Persistent workgroups of `waves_per_group` waves, no more than there are
// chunks for.  A batch too small to give half of the waves a chunk of 64
// reads is cut into smaller chunks, down to one read: a wave's time grows
// with its longest search and with the bytes it stages, so few reads a wave
// are done sooner (MI355X, 64 reads of 30-300 bases: 8 us as 64 chunks, 18 as
// one).  For all waves rather than half, launching them costs more than
// their smaller chunks save (100,000 reads of 25 bases: 13.0 against 10.0 us).
// A larger one is cut evenly: into as many reads a chunk as give every wave
// the same number of chunks, so that the last round of them is not nearly
// empty (4M reads: 11 rounds of 60 reads rather than 10 of 64 and a sixth of
// one).
inline SearchSplit search_split(int64_t nreads, int cus, int blocks_per_cu, int waves_per_group, int group) {
    const int64_t gmax = (int64_t)cus * blocks_per_cu, waves = gmax * waves_per_group;
    int per = 64;
    while (per > 1 && nreads / per < waves / 2) per /= 2;
    if (per == 64) {
        const int64_t rounds = (nreads + 64 * waves - 1) / (64 * waves);
        per = (int)((nreads + waves * rounds - 1) / (waves * rounds));
    }
    const int64_t chunks = (nreads + per - 1) / per;
    group = (int)std::max<int64_t>(1, std::min<int64_t>(group, chunks / gmax));
    // a workgroup has a block for itself, and a chunk for each wave
    const int64_t least = std::max(group, waves_per_group);
    return SearchSplit{per, chunks, group, (unsigned)std::min<int64_t>(gmax, (chunks + least - 1) / least)};
}

}  // namespace samatch
