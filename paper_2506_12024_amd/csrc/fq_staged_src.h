// Which stages of a stage-ordered plan need no grid barrier: plain code, so that a host program can check it against the
// rule written out.
//
// A stage's workgroups may start as soon as the x they read is written if every x of the stage lies in the y of one
// entry of the stage just before it; src[e] is then that entry's number + 1, and 0 for the entries of every other
// stage.  All or nothing for a plan: only if no two ys overlap, and every x lies in one y of an earlier stage or meets
// none, does what is read as x stay as its producer left it, and has every word that is waited for one writer
// (buffers used again for a later y go through the barrier).  Stages 0 and 1 never: the barrier behind stage 0
// is also the one that has every y cleared.  Nor a stage that reads an entry of which, at some of the widths that its
// stage may be switched to, a workgroup could be dealt more rows than it holds results for: that share is refused, its
// rows keep what they held, and nobody may wait for them.
#ifndef FQ_STAGED_SRC_H
#define FQ_STAGED_SRC_H

#include <algorithm>
#include <cstdint>
#include <vector>

#ifdef __HIPCC__
#define FQ_STAGED_FN __host__ __device__ inline
#else
#define FQ_STAGED_FN inline
#endif

// Relative cost of one row of one quantization group at each width (the one-launch kernel's table).
FQ_STAGED_FN int staged_group_cost(int bits)
{
    return bits == 2    ? 64 * 230 * 730 / 1000
           : bits == 3  ? 64 * 230 * 950 / 1000
           : bits == 4  ? 64 * 230
           : bits == 8  ? 128 * 200
           : bits == 16 ? 256 * 200
                        : 0;
}

// Chunks of 4 rows in the largest share of entry e of the stage [begin, end) at any of its entries' widths (a set of
// them: bit 0 .. 4 for 2, 3, 4, 8 and 16 bits).  The kernel deals `grid` workgroups to a stage: one to every entry, the
// others by cost, so e has at least 1 + floor(others x its part of the cost), its part being least at its cheapest width
// beside everyone else's dearest.
inline long long staged_largest_share(int e, int begin, int end, const int *K, const int *N, const int *widths, int grid)
{
    auto cost = [&](int i, bool most) {
        long long group = 0;
        for (int w = 0; w < 5; w++)
            if (widths[i] >> w & 1) {
                const long long c = staged_group_cost(w < 3 ? w + 2 : 8 << (w - 3));
                group = group == 0 || (c > group) == most ? c : group;
            }
        return group * (K[i] >> 7) * ((N[i] + 3) >> 2);
    };
    const long long own = cost(e, false), chunks = (N[e] + 3) >> 2;
    long long all = own;
    for (int i = begin; i < end; i++)
        if (i != e)
            all += cost(i, true);
    if (own == 0)
        return chunks;
    const long long workgroups = 1 + (grid - (end - begin)) * own / all;
    return (chunks + workgroups - 1) / workgroups;
}

// x[e], y[e]: address of the entry's first half; K[e], N[e]: how many; widths[e]: its copies; begin[s]: the first entry of stage
// s, begin[n_stages] = count; grid: workgroups of a launch; most: chunks of 4 rows a workgroup holds results for.
inline void staged_sources(int count, const uintptr_t *x, const uintptr_t *y, const int *K, const int *N, const int *widths,
                           const int32_t *stage, const int32_t *begin, int n_stages, int grid, int most, int32_t *src)
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
            all = all && from[e] >= begin[s - 1] &&
                  staged_largest_share(from[e], begin[s - 1], begin[s], K, N, widths, grid) <= most;
        for (int e = begin[s]; all && e < begin[s + 1]; e++)
            src[e] = from[e] + 1;
    }
}

#endif
