// CPU check of the rows that a wave looks at together while the prefix table
// is built (pivot.h), at the ends of the supported range of text lengths,
// built with the undefined-behaviour sanitizer.
#include <algorithm>
#include <cstdint>
#include <cstdio>

#include "pivot.h"

static int failures = 0;

static void fail(const char *what, int64_t lo, int64_t hi, int lane, int64_t got) {
    std::printf("%s: rows [%lld, %lld), lane %d: %lld\n", what, (long long)lo, (long long)hi, lane, (long long)got);
    failures++;
}

// What the lanes look at in [lo, hi): in range (or no row), in ascending order.
static void expect(int64_t lo, int64_t hi) {
    int64_t before = lo - 1;
    for (int lane = 0; lane < 64; lane++) {
        const int64_t got = samatch::wave_probe_row(lo, hi, lane);
        if (got < lo || (hi - lo > 64 && got >= hi)) fail("outside", lo, hi, lane, got);
        if (hi - lo <= 64 && got != lo + lane) fail("not its row", lo, hi, lane, got);
        if (got <= before) fail("not ascending", lo, hi, lane, got);
        before = got;
    }
}

// The first of n rows that is not below `target`, narrowed down as the kernel does.
static int64_t search(int64_t n, int64_t target) {
    uint32_t lo = 0, hi = (uint32_t)n;
    for (int turn = 0; lo < hi; turn++) {
        if (turn > 40) return -1;
        const int probes = (int)std::min<uint32_t>(hi - lo, 64);
        int to = probes;
        for (int lane = probes - 1; lane >= 0; lane--)
            if ((int64_t)samatch::wave_probe_row(lo, hi, lane) >= target) to = lane;
        const uint32_t above = samatch::wave_probe_row(lo, hi, std::min(to, 63));
        const uint32_t below = samatch::wave_probe_row(lo, hi, std::max(to - 1, 0));
        if (to < probes) hi = above;
        if (to > 0) lo = below + 1;
    }
    return lo;
}

int main() {
    const int64_t n = INT32_MAX;  // the largest text the index accepts
    for (int64_t rows : {1, 2, 63, 64, 65, 66, 127, 128, 129, 4097, 1 << 20}) {
        expect(0, rows);
        expect(n - rows, n);
    }
    expect(0, n);
    for (int64_t target : {(int64_t)0, (int64_t)1, n / 2, n - 66, n - 65, n - 64, n - 63, n - 2, n - 1, n})
        if (search(n, target) != target) fail("search", 0, n, 0, target);
    std::printf("%s\n", failures ? "FAIL" : "ok");
    return failures ? 1 : 0;
}
