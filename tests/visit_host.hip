// Host model of a wide traversal's node visits (compiled and run by
// test_visit_termination.py): the children that a visit reports met are
// stacked and visited in turn, as the kernels do, in a tree whose nodes have
// empty child slots.  Prints, per layout and ray, whether the ray is taken
// for finite, the nodes visited and the empty slots met.
#include <cstdio>
#include <cstring>

#include "traverse.h"

using namespace bvhlib;

namespace {

// Two nodes: the root has one leaf and node 1, node 1 two leaves.
void fill(bvh_node_bvh4 *n) {
    for (int i = 0; i < 2; i++) {
        std::memset(&n[i], 0, sizeof(n[i]));
        n[i].nchild = 2;
        for (int c = 0; c < 4; c++) {
            const bool on = c < 2;
            n[i].lo_x[c] = n[i].lo_y[c] = n[i].lo_z[c] = on ? (float)c : INFINITY;
            n[i].hi_x[c] = n[i].hi_y[c] = n[i].hi_z[c] = on ? (float)c + 0.5f : -INFINITY;
            n[i].child[c] = !on ? kRefEmpty : (i == 0 && c == 1 ? ref_interior(1) : ref_leaf((uint32_t)(i + c), 1));
        }
    }
}

template <class Node, class Q>
void fill8(Node *n, Q top) {
    for (int i = 0; i < 2; i++) {
        std::memset(&n[i], 0, sizeof(n[i]));
        n[i].nchild = 2;
        for (int a = 0; a < 3; a++) n[i].scale[a] = 1.5f / (float)top;
        for (int c = 0; c < 8; c++) {
            const bool on = c < 2;
            n[i].qlo_x[c] = n[i].qlo_y[c] = n[i].qlo_z[c] = on ? 0 : top;
            n[i].qhi_x[c] = n[i].qhi_y[c] = n[i].qhi_z[c] = on ? top : 0;
            n[i].child[c] = !on ? kRefEmpty : (i == 0 && c == 1 ? ref_interior(1) : ref_leaf((uint32_t)(i + c), 1));
        }
    }
}

template <class Dec>
void visit(const char *layout, const void *nodes, const char *name, const bvh_ray &ray) {
    const Ray r = load_ray(&ray, 0, 2.0f);
    const typename Dec::Prep prep = Dec::prep(r);
    uint32_t stack[64], sp = 0, visits = 0, empty = 0;
    stack[sp++] = ref_interior(0);
    while (sp > 0 && visits < 1000) {
        const uint32_t at = stack[--sp];
        if (!(at & 1u)) continue;
        u32x4 m[Dec::kWords];
        float tn[Dec::K];
        uint32_t ref[Dec::K];
        Dec::fetch(nodes, (at >> 1) < 1u ? (at >> 1) : 1u, prep, m);  // the kernels' index clamp
        visits++;
        if (r.fast) Dec::template test<true>(m, r, INFINITY, tn, ref);
        else Dec::template test<false>(m, r, INFINITY, tn, ref);
        for (int c = 0; c < Dec::K; c++) {
            if (tn[c] == INFINITY) continue;
            empty += ref[c] == kRefEmpty;
            if (sp < 64) stack[sp++] = ref[c];
        }
    }
    std::printf("%s %s finite %d visits %u empty %u\n", layout, name, (int)ray_finite(r), visits, empty);
}

}  // namespace

int main() {
    alignas(128) static bvh_node_bvh4 n4[2];
    alignas(128) static bvh_node_bvh8_q8 n8[2];
    alignas(32) static bvh_node_bvh8_q16 n16[2];
    fill(n4);
    fill8<bvh_node_bvh8_q8, uint8_t>(n8, 255);
    fill8<bvh_node_bvh8_q16, uint16_t>(n16, 65535);
    const float inf = INFINITY, nan = NAN;
    const struct {
        const char *name;
        alignas(16) bvh_ray r;
    } rays[] = {
        {"plain", {{-1, -1, -1}, 0, {1, 1, 1}, inf}},
        {"axis", {{0.25f, 0.25f, -1}, 0, {0, 0, 1}, inf}},
        {"no-direction", {{0.25f, 0.25f, 0.25f}, 0, {0, 0, 0}, inf}},
        {"nan-direction", {{0, 0, 0}, 0, {nan, nan, nan}, inf}},
        {"inf-direction", {{0, 0, 0}, 0, {inf, inf, inf}, inf}},
        {"minus-inf-direction", {{0, 0, 0}, 0, {-inf, -inf, -inf}, inf}},
        {"nan-origin", {{nan, nan, nan}, 0, {0, 0, 1}, inf}},
        {"inf-origin", {{inf, inf, inf}, 0, {1, 1, 1}, inf}},
        {"minus-inf-origin", {{-inf, -inf, -inf}, 0, {-1, 1, -1}, inf}},
        {"mixed", {{nan, 0, inf}, 0, {1, inf, nan}, inf}},
        {"huge", {{3e38f, -3e38f, 3e38f}, 0, {3e38f, 1e-45f, -3e38f}, inf}},
        {"nan-tmax", {{-1, -1, -1}, 0, {1, 1, 1}, nan}},
    };
    for (const auto &x : rays) {
        visit<DecodeBVH4>("bvh4", n4, x.name, x.r);
        visit<DecodeBVH8Q8>("bvh8_q8", n8, x.name, x.r);
        visit<DecodeBVH8Q16>("bvh8_q16", n16, x.name, x.r);
    }
    return 0;
}
