// Finishing a wave's last rays (or point queries) together.
//
// A persistent wave that finds no more rays to claim is left with its longest
// ones, and a launch of few rays gives every wave only a few from the start.
// Either way most lanes would idle while one lane walks a tree whose every
// step waits for memory: without the longest 0.1 % of them, 1 M closest-point queries
// on a 500 K-triangle sphere cluster took 2.1 ms instead of 3.2, and 1,000
// rays took as long as 30,000.  Here the lanes of the wave are shared out among
// the rays that are left (16 at most): a group of 64 / rays lanes takes
// the nearest entries of its ray's stack, one per lane, visits them at once,
// and stacks all their children.  Nodes that the plain order would have culled
// by then are visited in vain, in lanes that had nothing to do.  Every node
// that the best hit does not cull is visited in both orders, so the results
// are the same.
// Measured before and after (BVH4, uniform rays, the same scene): 1,000 rays
// 378 -> 30 us, 30,000 441 -> 98, 262,144 366 now, 1 M closest hits 1.29 ->
// 1.17 ms; terrain bounce rays 511 -> 447 us.
#pragma once

#include "traverse.h"

namespace bvhlib {

// How a launch deals its rays: `claim` to a wave at a time; a wave finishes
// its last `items` in groups of lanes, each keeping `reserve` entries of its
// stack free for going depth first.
struct Deal {
    uint32_t claim, items, reserve;
};

// At most kCoopItems rays of a wave are finished in groups.  1 M uniform rays
// on the sphere cluster, BVH4 / AABB2 / BVH8-Q8 (a ring of 16 entries): 0.95 /
// 1.77 / 1.04 ms at 8, 0.93 / 1.68 / 1.02 at 16, 0.98 / 1.65 / 1.50 at 32
// (groups of two lanes have 32 entries, which 8-wide rays outgrow).
constexpr uint32_t kCoopItems = 16;

// Entries that going depth first needs on a tree whose stack bound is
// max_stack, with room for one more node's children.
constexpr uint32_t depth_first_reserve(int32_t max_stack) { return (uint32_t)max_stack + 8u; }

// The waves among which a launch's rays are spread: three of four for BVH8-Q16,
// whose 160-byte nodes fill the vector L1 with the lines of three waves per SIMD
// (three against four: terrain camera rays 14 % faster at 7,428 and 8 % at 70,000
// to 160,000, uniform rays 8 % at 10,000), but not where fewer waves would have
// more rays than they finish in groups from the start (65,536 uniform rays 22 %
// slower).  BVH8-Q8 does not gain (160,000: camera rays 10 % faster in three,
// shadow rays 7 % and uniform ones 3 % slower).
constexpr uint64_t spread_waves(int layout, uint64_t waves) {
    return layout == BVH_LAYOUT_BVH8_Q16 ? waves * 3 / 4 : waves;
}

// n rays or queries on a grid of `waves` resident waves, with a ring of sl
// entries per lane: a group of 64 / items lanes has sl * 64 / items entries,
// at least 48 of them beside its reserve.  spread: spread_waves().
inline Deal deal_of(uint64_t n, uint64_t waves, int sl, uint32_t reserve, uint64_t spread) {
    Deal d;
    d.reserve = reserve;
    d.items = kCoopItems;
    while (d.items > 0 && 64u * (uint32_t)sl / d.items < reserve + 48u) d.items >>= 1;
    const auto share = [n](uint64_t w) {
        return (uint32_t)std::min<uint64_t>(64, std::max<uint64_t>(1, (n + w - 1) / w));
    };
    const auto kind = [&](uint32_t claim) { return claim <= d.items ? 0 : (claim <= kCoopItems ? 1 : 2); };
    d.claim = share(waves);
    if (kind(share(spread)) == kind(d.claim)) d.claim = share(spread);
    return d;
}

// A launch whose waves get one chunk each, of no more items than they finish
// in groups from the start, with a reserve that the tree's bound cannot
// exceed: no item can be left to the fallback pass, and no queue is read, so
// the launch needs neither that pass nor a cleared header.  Each is a launch
// that few rays notice: 1,000 rays without allocation 23.8 -> 21.0 us, 10,007
// closest points 34 -> 30 us.  More items per wave have no room for such a
// reserve (kRayReserve says what it costs) and take both launches.
inline bool wholly_coop(const Deal &d, uint64_t n, uint64_t waves, int32_t max_stack) {
    return n <= waves * d.claim && d.claim <= d.items && d.reserve >= depth_first_reserve(max_stack);
}
// Few rays need more entries than this at once (one that does is re-traced by
// the fallback pass); a reserve of the tree's worst case (some 60 entries)
// leaves 8 groups per wave instead of 16: 65,536 rays 159 -> 237 us.
constexpr uint32_t kRayReserve = 16;

// The smallest value of x in the calling lane's group of 1 << lg lanes.
__device__ inline float group_min(float x, uint32_t lg) {
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t d = 0; d < lg; d++) x = fminf(x, lane_f(x, lane ^ (1u << d)));
    return x;
}

// What a wave works on is a policy F:
//   Entry, kChildren           stack entry, children of a node at most
//   Best                       result so far: a metric (smaller is better), u, v, id
//   metric(best)
//   load(item)                 takes up ray or query `item` (an index)
//   cull(metric)               bound beyond which entries are skipped
//   breadth(metric, lanes)     entries to take at a time, at most
//   expand(entry, cull, kids, n, first, cnt)   the entry's unculled children,
//                              nearest first, or its leaf's triangles
//   leaves(want, first, cnt, best, wl)         tests the lanes' leaves; true
//                              in a lane that needs no more (every lane calls it)
//   store(item, best)          the result
//   list(item)                 to the fallback pass; false where none follows
//
// Called by every lane of the wave (converged); lanes whose item is not
// kNoRay hold one under way, at least one and at most kCoopItems of them.
// Their stacks lie wholly in the LDS ring, `entries` entries from its first
// slot on, the entry to visit next on top.  A group takes fewer entries at a
// time as its stack fills, down to one, which is the depth-first order that
// `reserve` entries suffice for.
template <class F, int SL>
__device__ inline void coop_finish(F &f, typename F::Entry *stack, uint32_t item, uint32_t entries,
                                   typename F::Best best, uint32_t reserve, WaveLeafLds *wl) {
    using E = typename F::Entry;
    constexpr int K = F::kChildren;
    constexpr uint32_t kMinGroup = 64u / kCoopItems;
    const uint32_t lane = threadIdx.x & 63u, wave0 = threadIdx.x & ~63u;
    // column of a lane of this wave in the ring
    auto slot = [&](uint32_t level, uint32_t of) -> E & { return stack[level * kTraceBlock + wave0 + of]; };

    // groups of 1 << lg lanes; group g takes the item of the g-th lane that has one
    const uint64_t busy = __builtin_amdgcn_ballot_w64(item != kNoRay);
    const uint32_t count = (uint32_t)__builtin_popcountll(busy);
    const uint32_t lg = 6u - (count > 1u ? 32u - (uint32_t)__builtin_clz(count - 1u) : 0u);
    const uint32_t g = lane >> lg, c = lane & ((1u << lg) - 1u);
    const uint64_t group = (lg == 6u ? ~0ull : (1ull << (1u << lg)) - 1ull) << (g << lg);
    if (item != kNoRay) wl->owner[count_below(busy)] = lane;
    wave_lds_sync();
    const bool live = g < count;
    const uint32_t own = wl->owner[live ? g : 0u];
    item = lane_u(item, own);
    const uint32_t of_own = lane_u(entries, own);
    uint32_t sp = live ? of_own : 0u;
    float metric = lane_f(F::metric(best), own);
    F::metric(best) = metric;
    best.u = lane_f(best.u, own);
    best.v = lane_f(best.v, own);
    best.id = lane_u(best.id, own);
    // entry e of a group's stack lies in level e >> lg of lane e mod (1 << lg)
    // of the group: every lane reads the entries that will be in its column
    // before any lane writes
    constexpr uint32_t kMine = (SL + kMinGroup - 1) / kMinGroup;
    E mine[kMine];
#pragma unroll
    for (uint32_t j = 0; j < kMine; j++) {
        const uint32_t e = (j << lg) + c;
        if (e < sp) mine[j] = slot(e, own);
    }
    wave_lds_sync();
#pragma unroll
    for (uint32_t j = 0; j < kMine; j++)
        if ((j << lg) + c < sp) slot(j, lane) = mine[j];
    wave_lds_sync();

    f.load(item);
    const uint32_t cap = (uint32_t)SL << lg;
    bool over = false;
    while (__builtin_amdgcn_ballot_w64(sp > 0) != 0) {
        // take as many entries as there are lanes, and as leave the reserve
        // free after K children each, but at least one
        const uint32_t room = cap - sp, spare = room > reserve ? room - reserve : 0u;
        const uint32_t k = min(min(sp, f.breadth(metric, 1u << lg)), max(spare / (uint32_t)(K - 1), 1u));
        const bool full = sp > 0 && room < (uint32_t)(K - 1);  // the reserve prevents it
        over = over || full;
        sp = full ? 0u : sp;
        E e[K];
        uint32_t n = 0, first = 0, cnt = 0;
        if (c < k && !full) {
            const uint32_t at = sp - 1u - c;
            const E x = slot(at >> lg, (g << lg) + (at & ((1u << lg) - 1u)));
            f.expand(x, f.cull(metric), e, n, first, cnt);
        }
        sp -= full ? 0u : k;
        // the children: those of the lanes with the nearest entries on top
        uint32_t below = 0, total = 0;
#pragma unroll
        for (int b = 0; (1 << b) <= K; b++) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(((n >> b) & 1u) != 0u) & group;
            below += count_below(m) << b;
            total += (uint32_t)__builtin_popcountll(m) << b;
        }
        wave_lds_sync();
        const uint32_t top = sp + total - below - 1u;  // the lane's nearest child
#pragma unroll
        for (int i = 0; i < K; i++) {
            const uint32_t at = top - (uint32_t)i;
            if ((uint32_t)i < n) slot(at >> lg, (g << lg) + (at & ((1u << lg) - 1u))) = e[i];
        }
        sp += total;
        if (__builtin_amdgcn_ballot_w64(cnt > 0) != 0) {
            const bool ended = f.leaves(cnt > 0, first, cnt, best, wl);
            if ((__builtin_amdgcn_ballot_w64(ended) & group) != 0) sp = 0;
            metric = group_min(F::metric(best), lg);
        }
        wave_lds_sync();
    }
    // the group's (metric, id) lexicographic best (metrics are never negative)
    const uint64_t key = (uint64_t)__float_as_uint(F::metric(best)) << 32 | best.id;
    uint64_t least = key;
    for (uint32_t d = 0; d < lg; d++) {
        const uint64_t other = (uint64_t)lane_u((uint32_t)(least >> 32), lane ^ (1u << d)) << 32 |
                               lane_u((uint32_t)least, lane ^ (1u << d));
        least = other < least ? other : least;
    }
    const uint64_t winners = __builtin_amdgcn_ballot_w64(key == least) & group;
    if (live && lane == (uint32_t)__builtin_ctzll(winners)) {
        // a launch without a fallback pass has the reserve that rules `over` out
        // (wholly_coop); were it reached all the same, the best so far is stored
        if (!over || !f.list(item)) f.store(item, best);
    }
}

// Rays of one scene.
template <class Tr, int LeafMode, int Mode>
struct FinishRays {
    using Entry = typename Tr::Entry;
    using Best = bvhlib::Best;
    static constexpr int kChildren = Tr::kChildren;
    const void *nodes;
    int64_t n_nodes;
    const SceneData &ld;
    const bvh_ray *rays;
    bvh_hit *hits;
    const Fallback &fb;
    Ray r{};
    typename Tr::Prep prep{};
    bool fast = true;
    __device__ static float &metric(Best &b) { return b.t; }
    __device__ void load(uint32_t item) {
        r = load_ray(rays, item, ld.coord_max);
        prep = Tr::prep(r);
        fast = __builtin_amdgcn_ballot_w64(!r.fast) == 0;
    }
    __device__ float cull(float t) const {
        return (Mode == BVH_TRACE_ANY ? fminf(r.tmax, INFINITY) : fminf(t, r.tmax)) * kFarScale;
    }
    __device__ uint32_t breadth(float, uint32_t lanes) const { return lanes; }
    __device__ void expand(Entry x, float bound, Entry *kids, uint32_t &n, uint32_t &first,
                           uint32_t &cnt) const {
        uint32_t leaf = kRefEmpty;
        Tr::expand(nodes, n_nodes, ld, r, prep, fast, bound, x, kids, n, leaf);
        if (leaf != kRefEmpty) {
            first = leaf >> 5;
            cnt = ((leaf >> 1) & 0xFu) + 1u;
        }
    }
    __device__ bool leaves(bool want, uint32_t first, uint32_t cnt, Best &best, WaveLeafLds *wl) const {
        uint32_t ntri = 0;
        return wave_test_leaves<LeafMode, Mode>(ld, r, want, first, cnt, best, ntri, wl);
    }
    __device__ void store(uint32_t item, const Best &best) const { store_hit(hits, item, best); }
    __device__ bool list(uint32_t item) const { return fallback_append(fb, item); }
};

}  // namespace bvhlib
