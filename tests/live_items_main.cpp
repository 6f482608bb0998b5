// Host check of the batch programs' maps of live items (csrc/live_items.h):
// after a fill that failed between plan() and hold(), no set of patches counts
// as held; the spans cover each live item and cube once.  Exit status 0: all
// checks hold.
#include <cstdio>

#include "live_items.h"

static int bad = 0;
static void check(bool ok, const char *what) {
    if (!ok) {
        std::printf("FAILED %s\n", what);
        bad++;
    }
}

int main() {
    mg::LiveItems I;
    // two launches over three patches: a smoother (cubes allowed up to 8) and
    // one that always runs its items
    I.first = {100, 200};
    I.cube_max = {8, 0};
    I.cube_at = {40, 0};
    const int n[3] = {5, 3, 7}, cubes[3] = {4, 4, 8};
    int at[2] = {0, 0};
    for (int l = 0; l < 2; l++)
        for (int p = 0; p < 3; p++) {
            I.ranges.push_back({l, p, at[l], n[p], p * 16, p, cubes[p]});
            at[l] += n[p];
        }
    mg::Span out[12];
    const std::vector<char> all = {1, 1, 1}, two = {1, 1, 0}, none = {0, 0, 0};

    check(!I.holds(all) && !I.holds(none), "nothing held at first");
    int ns = I.plan(all, out);  // 16 cubes: above the launch's 8, items only
    check(ns == 6 && I.live_cubes[0] == -1 && I.live[0] == 15 && I.live[1] == 15, "all patches");
    check(!I.holds(all), "not held before the fill is enqueued");
    I.hold(all);
    check(I.holds(all) && !I.holds(two), "held after it");

    ns = I.plan(two, out);  // 8 cubes: over cubes
    check(ns == 6 && I.live_cubes[0] == 8 && I.live_cubes[1] == -1 && I.live[0] == 8, "two patches");
    check(out[0].lev == 0 && out[0].dst == 40 && out[0].n == 4 && out[2].lev == 16 && out[2].dst == 44, "cube spans");
    check(out[1].lev == -1 && out[1].src == 0 && out[1].dst == 100 && out[3].src == 5 && out[3].dst == 105,
          "item spans");
    // the fill failed here: neither the new set nor the old one is in the maps
    check(!I.holds(two), "a failed fill is planned again");
    check(!I.holds(all), "the set before it is no longer held");
    ns = I.plan(two, out);
    check(ns == 6 && I.live[0] == 8 && I.live_cubes[0] == 8, "planned again");
    I.hold(two);
    check(I.holds(two), "held after the second fill");

    ns = I.plan(none, out);
    check(ns == 0 && I.live[0] == 0 && I.live_cubes[0] == 0, "no patches");
    I.hold(none);
    check(I.holds(none), "an empty set can be held");
    std::printf("live items: %d failed\n", bad);
    return bad != 0;
}
