// Slices of a served query's task space (host only). The first tasks are shares of
// split roots, a root in `ways` tasks each; the rest are whole roots. Rates are
// kept in roots, so that a rate measured on shares says what whole roots take: counted in
// tasks, a slice that left the split roots took up to `ways` times its time.
#pragma once
#include <algorithm>
#include <cstdint>

namespace gpint {

struct TaskSplit {
    int64_t tasks = 0;  // tasks that are shares of split roots
    int ways = 1;       // shares of a root

    // Roots in tasks [first, first + n).
    double roots(int64_t first, int64_t n) const {
        const int64_t shares = std::max<int64_t>(0, std::min(first + n, tasks) - first);
        return (double)shares / ways + (double)(n - shares);
    }
    // Tasks from `first` on that hold so many roots.
    int64_t tasks_of(int64_t first, double roots) const {
        const double left = (double)std::max<int64_t>(0, tasks - first) / ways;
        const double n = roots <= left ? roots * ways : left * ways + (roots - left);
        return (int64_t)std::min(n, 1e12);
    }
};

// The next slice of a query, from task `next` on: its share of the target iteration
// (fair seconds) at the rate of a slice of n tasks from `first` that took `seconds`. The
// first roots are the heaviest, so the rate errs low: it may grow fast. total: the
// query's tasks (0: not known); a rest of up to two shares goes at once.
inline int64_t next_slice(const TaskSplit& split, int64_t first, int64_t n, double seconds, int64_t next, double fair,
                          int64_t total = 0) {
    const double roots = split.roots(first, n);
    const double want = std::min(roots / std::max(1e-7, seconds) * fair, 32.0 * roots + 1);
    if (next < total && split.roots(next, total - next) <= 2 * want) return total - next;
    return std::max<int64_t>(64, split.tasks_of(next, want));
}

}  // namespace gpint
