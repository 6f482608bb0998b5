// Host bookkeeping of a batch program's maps of live items (batch.hip): which
// patches the device maps hold, the spans that fill them for another set of
// patches, and each launch's live items and cubes.  No device code.
#pragma once

#include <vector>

namespace mg {

// `n` entries of one launch's map from place dst on: the positions src ..
// src + n - 1 of one patch's items or, with lev >= 0, that patch level's cubes
// (src: their selector).
struct Span {
    int src, dst, n, lev;
};

struct LiveItems {
    struct Range {  // one patch's items of one launch
        int launch, patch, first, n;
        int lev, sel, cubes;  // the items' level and selector; smoother launches: the level's cubes
    };
    std::vector<Range> ranges;
    std::vector<int> first;              // per launch: its items' place in the map
    std::vector<int> cube_max, cube_at;  // per launch: most live cubes it runs over (0: its items always), their place
    std::vector<int> live, live_cubes;   // per launch; live_cubes: -1 where it runs its items

    // Whether the device maps hold exactly the patches marked in `on`.
    bool holds(const std::vector<char> &on) const { return !mapped.empty() && mapped == on; }

    // The spans (at most two per range) that make the maps hold `on`, and the
    // counts that go with them.  From here to hold() the maps count as holding
    // nothing: where the copy or the kernel that fills them fails, the next
    // call plans anew instead of walking entries that were never written.
    int plan(const std::vector<char> &on, Span *out) {
        mapped.clear();
        const size_t nk = first.size();
        live.assign(nk, 0);
        live_cubes.assign(nk, 0);
        for (const Range &r : ranges)
            if (on[r.patch]) live_cubes[r.launch] += r.cubes;
        for (size_t i = 0; i < nk; i++) live_cubes[i] = cube_max[i] > 0 && live_cubes[i] <= cube_max[i] ? 0 : -1;
        int ns = 0;
        for (const Range &r : ranges)
            if (on[r.patch]) {
                const int i = r.launch;
                if (live_cubes[i] >= 0) {
                    out[ns++] = Span{r.sel, cube_at[i] + live_cubes[i], r.cubes, r.lev};
                    live_cubes[i] += r.cubes;
                }
                out[ns++] = Span{r.first, first[i] + live[i], r.n, -1};
                live[i] += r.n;
            }
        return ns;
    }
    // The maps have been enqueued for `on`, copy and kernel without an error.
    void hold(const std::vector<char> &on) { mapped = on; }

private:
    std::vector<char> mapped;  // empty: none
};

}  // namespace mg
