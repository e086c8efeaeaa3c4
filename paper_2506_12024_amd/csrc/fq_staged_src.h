// Which stages of a stage-ordered plan need no grid barrier: plain code, so that a host program can check it against the
// rule written out.
//
// A stage's workgroups may start as soon as the x they read is written if every x of the stage lies in the y of one
// entry of the stage just before it; src[e] is then that entry's number + 1, and 0 for the entries of every other
// stage.  All or nothing for a plan: only if no two ys overlap, and every x lies in one y of an earlier stage or meets
// none, does what is read as x stay as its producer left it, and has every word that is waited for one writer
// (buffers used again for a later y go through the barrier).  Stages 0 and 1 never: the barrier behind stage 0
// is also the one that has every y cleared.
#ifndef FQ_STAGED_SRC_H
#define FQ_STAGED_SRC_H

#include <algorithm>
#include <cstdint>
#include <vector>

// x[e], y[e]: address of the entry's first half; K[e], N[e]: how many; begin[s]: the first entry of stage s, begin[n_stages]
// = count.
inline void staged_sources(int count, const uintptr_t *x, const uintptr_t *y, const int *K, const int *N, const int32_t *stage,
                           const int32_t *begin, int n_stages, int32_t *src)
{
    std::vector<int> by(count), from(count, -1); // entries in the order of their ys; whose y an x lies in
    for (int e = 0; e < count; e++)
        by[e] = e, src[e] = 0;
    auto y_end = [&](int e) { return y[e] + 2 * (uintptr_t)N[e]; };
    std::sort(by.begin(), by.end(), [&](int a, int b) { return y[a] < y[b]; });
    for (int i = 1; i < count; i++)
        if (y_end(by[i - 1]) > y[by[i]])
            return;
    for (int e = 0; e < count; e++) {
        const uintptr_t x_end = x[e] + 2 * (uintptr_t)K[e];
        const auto after = std::upper_bound(by.begin(), by.end(), x[e], [&](uintptr_t v, int b) { return v < y[b]; });
        if (after != by.end() && y[*after] < x_end)
            return; // a y begins inside this x
        if (after == by.begin() || y_end(after[-1]) <= x[e])
            continue; // it meets none
        from[e] = after[-1];
        if (y_end(from[e]) < x_end || stage[from[e]] >= stage[e])
            return;
    }
    for (int s = 2; s < n_stages; s++) {
        bool all = true;
        for (int e = begin[s]; e < begin[s + 1]; e++)
            all = all && from[e] >= begin[s - 1];
        for (int e = begin[s]; all && e < begin[s + 1]; e++)
            src[e] = from[e] + 1;
    }
}

#endif
