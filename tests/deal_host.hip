// Host model of the stack that a group of lanes shares while it finishes a ray
// (compiled and run by test_deal_bounds.py).  For launches without a fallback
// pass, prints the least room that any group has left for a node's children on
// trees that use their stack bound to the full; then what the fallback list
// does where there is one and where there is none.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "coop.h"

using namespace bvhlib;

namespace {

// Room left before a node's K children are stacked, at least, over the first
// steps of a walk that culls nothing; every interior node has K children down
// to the depth that the bound allows.
int least_room(const Deal &d, int sl, uint32_t lanes, int K, int max_stack) {
    const int cap = sl * (int)lanes, depth = max_stack / (K - 1);
    std::vector<int> st(1, 0);  // entries: their depths, the nearest on top
    int least = cap;
    for (int step = 0; step < 3000 && !st.empty(); step++) {
        const int sp = (int)st.size(), room = cap - sp;
        const int spare = room > (int)d.reserve ? room - (int)d.reserve : 0;
        const int k = std::min(std::min(sp, (int)lanes), std::max(spare / (K - 1), 1));
        least = std::min(least, room - (K - 1));
        std::vector<int> taken(st.end() - k, st.end());
        st.resize(sp - k);
        for (int t : taken)
            if (t < depth) st.insert(st.end(), K, t + 1);
        if ((int)st.size() > cap) return -1;
    }
    return least;
}

}  // namespace

int main() {
    const uint64_t waves = 4096;
    for (int K : {2, 4, 8})
        for (int sl : {8, 16, 32})
            for (int max_stack : {0, 1, 7, 21, 40, 63, 100, 200, 256}) {
                int least = 1 << 30, launches = 0;
                const uint64_t spread = spread_waves(K == 8 ? BVH_LAYOUT_BVH8_Q16 : BVH_LAYOUT_BVH4, waves);
                for (uint32_t per = 1; per <= 17; per++) {
                    const uint64_t n = waves * per;
                    const Deal d = deal_of(n, waves, sl, depth_first_reserve(max_stack), spread);
                    if (!wholly_coop(d, n, waves, max_stack)) continue;
                    launches++;
                    for (uint32_t items = 1; items <= d.claim; items++) {
                        uint32_t lanes = 64;
                        while (64 / lanes < items) lanes /= 2;
                        least = std::min(least, least_room(d, sl, lanes, K, max_stack));
                    }
                }
                std::printf("%d %d %d %d %d\n", K, sl, max_stack, launches, least);
            }
    // the spill area of the launches that have one: runs for every lane that can
    // hold a ray, never fewer for more rays, and few more than rays
    int short_runs = 0, shrinking = 0;
    uint64_t before = 0, most = 0;
    for (uint64_t n = 1; n < 3 * 64 * waves; n += n < 100000 ? 1 : 37) {
        const uint64_t runs = spill_runs(n, waves / 4);
        for (uint64_t spread : {waves, waves * 3 / 4})
            for (uint32_t reserve : {kRayReserve, depth_first_reserve(256)}) {
                const Deal d = deal_of(n, waves, 16, reserve, spread);
                const uint64_t blocks = std::min<uint64_t>(waves / 4, ((n + d.claim - 1) / d.claim + 3) / 4);
                // spread thin: dealt in one round, as the kernels see it
                if (d.claim < 64 && n > blocks * 4 * d.claim) short_runs++;
                if (blocks * 4 * std::min(d.claim, 64u) > runs) short_runs++;
            }
        shrinking += runs < before;
        before = runs;
        most = std::max(most, runs > n ? runs - n : 0);
    }
    std::printf("runs %d %d %d\n", short_runs, shrinking, most <= 2 * kTraceBlock);

    // the list itself, with a fallback pass and without
    uint32_t count = 0, list[4] = {};
    Fallback fb{};
    fb.count = &count;
    fb.list = list;
    const bool with = fallback_append(fb, 5) && fallback_append(fb, 9);
    const bool without = fallback_append(Fallback{}, 7);
    std::printf("list %d %u %u %u %d\n", (int)with, count, list[0], list[1], (int)without);
    return 0;
}
