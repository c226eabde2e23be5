// Launch geometry, free of HIP so that it is tested on the host.
#pragma once

#include <cstdint>

namespace slg {

// HIP takes a launch only while workgroups * threads < 2^32: the most
// workgroups of `threads` threads (limit > 0: and at most that many).
constexpr int64_t max_workgroups(int threads, int64_t limit = 0) {
    const int64_t most = ((int64_t(1) << 32) - 1) / threads;
    return limit > 0 && limit < most ? limit : most;
}

// The hub tier's workgroups: every group of `rows` of the hub rows [lo, hi)
// with every window from first_window to the last of `kept` positions,
// window by window, `cap` of them per launch. The number of a workgroup is
// its launch's base plus its place in the launch: group number % groups,
// window first_window + number / groups. (3.0e6 kept rows in 186 windows are
// 1.8e7 counting workgroups, past a single launch's 8.4e6.)
struct HubGrid {
    int64_t groups, total, cap;
    HubGrid(int64_t lo, int64_t hi, int rows, int64_t kept, int window_bits, int64_t first_window, int threads,
            int64_t limit)
        : groups((hi - lo + rows - 1) / rows),
          total(groups * ((kept >> window_bits) + 1 - first_window)),
          cap(max_workgroups(threads, limit)) {}
    int64_t count(int64_t base) const { return total - base < cap ? total - base : cap; }
};

// Rows of N classes, the last class first, `rows0` of class 0 and `rows` of
// any other per workgroup, in launches of at most `cap` workgroups: next()
// takes the next launch's rows and returns its workgroups (0: none are left).
template <int N>
struct ClassRuns {
    int64_t begin[N] = {}, count[N] = {};  // this launch's rows of each class
    unsigned first[N] = {};                // first workgroup of class N - 1, ..., 0
    unsigned next(const int64_t *counts, int rows0, int rows, int64_t cap) {
        int64_t grid = 0;
        for (int r = 0; r < N; ++r) {
            const int c = N - 1 - r;
            const int64_t per = c ? rows : rows0, room = (cap - grid) * per;
            begin[c] += count[c];
            count[c] = counts[c] - begin[c] < room ? counts[c] - begin[c] : room;
            first[r] = (unsigned)grid;
            grid += (count[c] + per - 1) / per;
        }
        return (unsigned)grid;
    }
};

}  // namespace slg
