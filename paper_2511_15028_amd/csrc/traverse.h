// Device-side traversal shared by the per-scene and the batched kernels.
//
// One traversal routine per node family (binary nodes that carry their own
// box; wide nodes that carry their children's boxes), each instantiated with a
// layout decoder, so the search order and culling logic are written once and
// the node format is a type parameter: the decoupling of traversal from
// layout argued in Sec. 3-4 of the paper.
#pragma once

#include <cmath>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace bvhlib {


// Traversal kernels run 256 threads (four wave64) per block; the per-lane
// LDS stack columns are indexed by threadIdx.x with this stride.
constexpr int kTraceBlock = 256;

// Slab-test widening: far distances are scaled by 1 + 2^-21, above the
// 1 + 2 gamma_3 bound on the relative rounding error of (plane - o) * (1/d)
// (Ize 2013), so a box that the exact ray enters before the current best
// distance is never culled.
constexpr float kFarScale = 1.000000476837158203125f;

struct Ray {
    float ox, oy, oz;
    float dx, dy, dz;
    float rx, ry, rz;  // 1/d, IEEE (+-inf for +-0)
    float tmax;
    float knx, kny, knz;  // -(o * rdir) rounded up / down, for the one-FMA slab
    float kfx, kfy, kfz;  // distances (see slab_nf)
    bool nx, ny, nz;   // sign bits of d
    bool fast;         // the one-FMA slab distances are valid for this ray
};

// Scenes whose coordinates exceed this magnitude, and rays whose origin or
// 1/d components lie outside [2^-60, 2^60] in magnitude, use the two-rounding
// slab distances; everything else uses the one-FMA form.
constexpr float kFastLimit = 1.152921504606846976e18f;  // 2^60

// o * rdir moved outward by at least one ulp: the returned pair (lo, hi)
// brackets the exact product.
__host__ __device__ inline void bracket_product(float o, float rd, float &lo, float &hi) {
    const float c = o * rd;
    const float delta = fabsf(c) * 2.384185791015625e-07f + 2.350988701644575e-38f;  // 2^-22, 2^-125
    lo = c - delta;
    hi = c + delta;
}

// coord_max: largest coordinate magnitude of the scene (or +inf).
__host__ __device__ inline Ray load_ray(const bvh_ray *rays, uint64_t i, float coord_max) {
    const float4 *p = reinterpret_cast<const float4 *>(rays + i);
    const float4 a = p[0], b = p[1];
    Ray r;
    r.ox = a.x; r.oy = a.y; r.oz = a.z;
    r.dx = b.x; r.dy = b.y; r.dz = b.z;
    r.tmax = b.w;
    r.rx = 1.0f / r.dx;
    r.ry = 1.0f / r.dy;
    r.rz = 1.0f / r.dz;
    r.nx = __builtin_signbitf(r.dx);
    r.ny = __builtin_signbitf(r.dy);
    r.nz = __builtin_signbitf(r.dz);
    float lo, hi;
    bracket_product(r.ox, r.rx, lo, hi);
    r.knx = -hi; r.kfx = -lo;
    bracket_product(r.oy, r.ry, lo, hi);
    r.kny = -hi; r.kfy = -lo;
    bracket_product(r.oz, r.rz, lo, hi);
    r.knz = -hi; r.kfz = -lo;
    const float rmax = fmaxf(fabsf(r.rx), fmaxf(fabsf(r.ry), fabsf(r.rz)));
    const float rmin = fminf(fabsf(r.rx), fminf(fabsf(r.ry), fabsf(r.rz)));
    const float omax = fmaxf(fabsf(r.ox), fmaxf(fabsf(r.oy), fabsf(r.oz)));
    r.fast = rmax <= kFastLimit && rmin >= 1.0f / kFastLimit && omax <= kFastLimit &&
             coord_max <= kFastLimit;  // false for NaN as well
    return r;
}

// False for a ray with a NaN or infinite origin or direction component: the
// ray/triangle test accepts nothing for it (det, or one of U, V and T, is not
// finite), while its NaN slab distances cull no box.
__host__ __device__ inline bool ray_finite(const Ray &r) {
    const float z = r.ox * 0.0f + r.oy * 0.0f + r.oz * 0.0f + r.dx * 0.0f + r.dy * 0.0f + r.dz * 0.0f;
    return z == 0.0f;
}

// True when every active lane's ray can use the one-FMA slab distances (a
// wave-uniform value, so the choice costs one scalar branch).
__device__ inline bool wave_fast(const Ray &r) {
    return __builtin_amdgcn_ballot_w64(!r.fast) == 0;
}

// True when the rays of the lanes in `mask` (those with `has` set) all point
// into the same octant.  Called by every lane of the wave, so the result is
// wave-uniform.
__device__ inline bool rays_share_octant(const Ray &r, bool has, uint64_t mask) {
    const uint64_t nx = __builtin_amdgcn_ballot_w64(has && r.nx);
    const uint64_t ny = __builtin_amdgcn_ballot_w64(has && r.ny);
    const uint64_t nz = __builtin_amdgcn_ballot_w64(has && r.nz);
    return (nx == 0 || nx == mask) && (ny == 0 || ny == mask) && (nz == 0 || nz == mask);
}

// Ray/box test (the slab method of Kay and Kajiya; the paper's traversal
// tests node boxes with it, App. G) on planes already ordered by the ray:
// (nx, ny, nz) are the planes the ray enters through (the lower plane of an
// axis where d >= +0, the upper where d <= -0), (fx, fy, fz) the planes it
// leaves through.  The node cull is folded in: the far end is
// clipped at tcur (the best hit so far, or tmax).  Returns the entry
// distance, or +inf when the box is culled.
//
// Plane distances: the two-rounding form (plane - o) * rdir, or, when Fast, one FMA plane * rdir - o * rdir with the product o * rdir
// bracketed outward (entry planes subtract an upper bound, exit planes a
// lower bound), so the computed entry distance never exceeds
// (plane - o) * rdir by more than one rounding and the exit distance never
// falls short of it by more than one rounding.  Either way the relative
// error of each distance against the exact (plane - o) / d stays below the
// far-distance widening, so no box that the ray meets before the best hit is culled.
template <bool Fast>
__host__ __device__ inline float slab_nf(const Ray &r, float nx, float ny, float nz, float fx, float fy,
                                float fz, float cull) {
    float tnx, tny, tnz, tfx, tfy, tfz;
    if (Fast) {
        tnx = fmaf(nx, r.rx, r.knx); tfx = fmaf(fx, r.rx, r.kfx);
        tny = fmaf(ny, r.ry, r.kny); tfy = fmaf(fy, r.ry, r.kfy);
        tnz = fmaf(nz, r.rz, r.knz); tfz = fmaf(fz, r.rz, r.kfz);
    } else {
        tnx = (nx - r.ox) * r.rx; tfx = (fx - r.ox) * r.rx;
        tny = (ny - r.oy) * r.ry; tfy = (fy - r.oy) * r.ry;
        tnz = (nz - r.oz) * r.rz; tfz = (fz - r.oz) * r.rz;
    }
    const float t_near = fmaxf(0.0f, fmaxf(tnx, fmaxf(tny, tnz)));
    const float t_far = fminf(tfx, fminf(tfy, tfz)) * kFarScale;
    return (t_near <= fminf(cull, t_far)) ? t_near : INFINITY;
}

// The same test on a box given as (lo, hi): the entry and exit planes are
// chosen by the sign bit of each direction component.
template <bool Fast>
__device__ inline float slab(const Ray &r, float lox, float loy, float loz, float hix, float hiy,
                             float hiz, float cull) {
    return slab_nf<Fast>(r, r.nx ? hix : lox, r.ny ? hiy : loy, r.nz ? hiz : loz,
                         r.nx ? lox : hix, r.ny ? loy : hiy, r.nz ? loz : hiz, cull);
}

// Ray/triangle test: Moller and Trumbore (1997), with App. G's acceptance
// intervals (u, v >= 0 and u + v <= 1 inclusive, both faces; 0 < t <= tmax).
// Given p0 and the edges e1 = p1 - p0, e2 = p2 - p0 (as stored in a
// compacted leaf record), the hit o + t d = p0 + u e1 + v e2 is solved by
// Cramer's rule through P = d x e2, det = e1 . P, S = o - p0, Q = S x e1:
// U = S . P, V = d . Q, T = e2 . Q are u, v, t times det.  The interval
// tests run on those numerators with det's sign bit moved onto them (exact),
// against |det|, so only an accepted hit pays for the one correctly rounded
// division: t, u, v = (T, U, V) * (1 / |det|).  Every cross-product
// component is one product and one fused multiply-add, every dot product
// one product and two fused multiply-adds, in a fixed order, so the results
// are a fixed function of the f32 inputs (30 VALU operations up to the
// tests).
struct TriNum {
    float U, V, T, adet;
};

// The numerators and |det| of the test (no acceptance decision).
__device__ inline TriNum tri_numerators(const Ray &r, float p0x, float p0y, float p0z, float e1x,
                                        float e1y, float e1z, float e2x, float e2y, float e2z) {
    const float px = fmaf(r.dy, e2z, -(r.dz * e2y));
    const float py = fmaf(r.dz, e2x, -(r.dx * e2z));
    const float pz = fmaf(r.dx, e2y, -(r.dy * e2x));
    const float det = fmaf(e1z, pz, fmaf(e1y, py, e1x * px));
    const uint32_t sgn = __float_as_uint(det) & 0x80000000u;
    const float sx = r.ox - p0x, sy = r.oy - p0y, sz = r.oz - p0z;
    const float qx = fmaf(sy, e1z, -(sz * e1y));
    const float qy = fmaf(sz, e1x, -(sx * e1z));
    const float qz = fmaf(sx, e1y, -(sy * e1x));
    TriNum n;
    n.U = __uint_as_float(__float_as_uint(fmaf(sz, pz, fmaf(sy, py, sx * px))) ^ sgn);
    n.V = __uint_as_float(__float_as_uint(fmaf(r.dz, qz, fmaf(r.dy, qy, r.dx * qx))) ^ sgn);
    n.T = __uint_as_float(__float_as_uint(fmaf(e2z, qz, fmaf(e2y, qy, e2x * qx))) ^ sgn);
    n.adet = fabsf(det);
    return n;
}

__device__ inline bool tri_accept(const TriNum &n, float tmax) {
    return n.adet > 0.0f && n.adet < INFINITY && n.U >= 0.0f && n.V >= 0.0f &&
           n.U + n.V <= n.adet && n.T > 0.0f && n.T <= n.adet * tmax;
}

__device__ inline bool mt_edges(const Ray &r, float p0x, float p0y, float p0z, float e1x,
                                float e1y, float e1z, float e2x, float e2y, float e2z, float &t,
                                float &u, float &v) {
    const TriNum n = tri_numerators(r, p0x, p0y, p0z, e1x, e1y, e1z, e2x, e2y, e2z);
    if (!tri_accept(n, r.tmax)) return false;
    const float inv = 1.0f / n.adet;
    t = n.T * inv;
    u = n.U * inv;
    v = n.V * inv;
    return true;
}

// The same test from the three vertices.
__device__ inline bool mt(const Ray &r, float p0x, float p0y, float p0z, float p1x, float p1y,
                          float p1z, float p2x, float p2y, float p2z, float &t, float &u,
                          float &v) {
    return mt_edges(r, p0x, p0y, p0z, p1x - p0x, p1y - p0y, p1z - p0z, p2x - p0x, p2y - p0y,
                    p2z - p0z, t, u, v);
}

struct Best {
    float t, u, v;
    uint32_t id;  // 0xFFFFFFFF = none (compares above every valid id)
};

// (t, id) lexicographic improvement: lower t, then lower primitive id.
__device__ inline void consider(Best &b, float t, float u, float v, uint32_t id) {
    if (t < b.t || (t == b.t && id < b.id)) {
        b.t = t;
        b.u = u;
        b.v = v;
        b.id = id;
    }
}

// Per-scene data the kernels need besides the node buffer.  Leaf storage:
// COMPACT reads 48-B records {p0, e1 = p1 - p0, e2 = p2 - p0, prim id} in
// leaf order; INDEXED
// reads a primitive id, its three vertex indices and three vertices.
struct SceneData {
    const void *leaf;
    const float *verts;
    const int32_t *tris;
    uint32_t n_tris;
    float coord_max;  // largest coordinate magnitude of the scene (selects the slab form)
    float fo[3], fs[3];  // PBRT_Q16, SG_EQ: lower plane = fmaf(q, fs[a], fo[a])
    float ft[3];         // SG_EQ: upper plane = fmaf(-q, fs[a], ft[a])
    const void *topo;    // split layouts: the topology array after the boxes
};

// Compacted leaves: triangles are fetched in batches of kLeafBatch (all loads
// issued before the first test, so their latencies overlap).
constexpr uint32_t kLeafBatch = 4;

// Tests triangles [first, first+n) of the leaf order.  Returns true when an
// any-hit query is satisfied.
template <int LeafMode, int Mode>
__device__ inline bool test_leaf(const SceneData &ld, const Ray &r, uint32_t first, uint32_t n,
                                 Best &best, uint32_t &ntri) {
    const uint32_t end = min(first + n, ld.n_tris);  // bounds guard; a valid tree never clips
    if (LeafMode == BVH_LEAF_COMPACT) {
        const float4 *base = static_cast<const float4 *>(ld.leaf);
        for (uint32_t k0 = first; k0 < end; k0 += kLeafBatch) {
            float4 qa[kLeafBatch], qb[kLeafBatch];
            float2 qc[kLeafBatch];  // e2.z and the prim id (the record's padding is not read)
#pragma unroll
            for (uint32_t j = 0; j < kLeafBatch; j++) {
                if (k0 + j < end) {
                    const float4 *p = base + 3 * (size_t)(k0 + j);
                    qa[j] = p[0];
                    qb[j] = p[1];
                    qc[j] = *reinterpret_cast<const float2 *>(p + 2);
                }
            }
            bool found = false;
#pragma unroll
            for (uint32_t j = 0; j < kLeafBatch; j++) {
                if (k0 + j < end && !found) {
                    ntri++;
                    float t, u, v;
                    const float4 a = qa[j], b = qb[j];
                    const float2 c = qc[j];
                    if (mt_edges(r, a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, t, u, v)) {
                        consider(best, t, u, v, __float_as_uint(c.y));
                        found = Mode == BVH_TRACE_ANY;
                    }
                }
            }
            if (found) return true;
        }
        return false;
    }
    for (uint32_t k = first; k < end; k++) {
        const uint32_t id = (uint32_t) static_cast<const int32_t *>(ld.leaf)[k];
        const int32_t *tv = ld.tris + 3 * (size_t)id;
        const float *a = ld.verts + 3 * (size_t)tv[0];
        const float *b = ld.verts + 3 * (size_t)tv[1];
        const float *c = ld.verts + 3 * (size_t)tv[2];
        ntri++;
        float t, u, v;
        if (mt(r, a[0], a[1], a[2], b[0], b[1], b[2], c[0], c[1], c[2], t, u, v)) {
            consider(best, t, u, v, id);
            if (Mode == BVH_TRACE_ANY) return true;
        }
    }
    return false;
}

// ---------------------------------------------------------------------------
// Wave-level leaf batching: the lanes of a wave that hold a leaf to test
// publish its triangles, and the wave tests the (ray, triangle) pairs one per
// lane, so a leaf phase costs one triangle test per 64 pairs instead of one
// per triangle of the largest leaf.  Per round of up to 64 pairs:
//   * pair slots are assigned by an exclusive prefix sum of the leaf sizes
//     over the lanes (five ballots: leaf sizes are below 32);
//   * each leaf lane writes its lane number into the slots of its pairs (an
//     LDS table), each pair lane reads its owner and fetches the owner's ray
//     and leaf start from the owner's registers (ds_bpermute);
//   * hits are reduced per owner with an LDS 64-bit minimum of
//     (t bits << 32 | primitive id): t > 0, so the bits order like the
//     values, and the minimum is the (t, id) lexicographic best; the lane
//     holding that pair then stores its (u, v) for the owner.
// The arithmetic of each test is exactly that of test_leaf, so the hits are
// the same bits.
// ---------------------------------------------------------------------------
struct WaveLeafLds {
    unsigned long long key[64];  // per owner lane: best (t bits, id) of the round
    float2 uv[64];               // per owner lane: (u, v) of that best
    uint32_t owner[64];          // per pair slot of the round: owner lane
};
constexpr int kWavesPerBlock = kTraceBlock / 64;

// Orders the calling wave's LDS accesses on either side (a wave executes
// its LDS instructions in order; this keeps the compiler from moving them).
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Set bits of m below the calling lane.
__device__ inline uint32_t count_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ inline float lane_f(float x, uint32_t src) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute((int)(src << 2), __float_as_int(x)));
}
__device__ inline uint32_t lane_u(uint32_t x, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)x);
}

// Called by every lane of the wave (converged).  Lanes with `want` set test
// triangles [first, first + cnt) of the leaf order against their ray; their
// best is updated and their triangle counter advanced.  Returns true in a
// want lane whose any-hit query was satisfied.
template <int LeafMode, int Mode>
__device__ inline bool wave_test_leaves(const SceneData &ld, const Ray &r, bool want,
                                        uint32_t first, uint32_t cnt, Best &best, uint32_t &ntri,
                                        WaveLeafLds *wl) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t c = want ? cnt : 0u;
    uint32_t pre = 0, total = 0;
#pragma unroll
    for (int b = 0; b < 5; b++) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(((c >> b) & 1u) != 0u);
        pre += count_below(m) << b;
        total += (uint32_t)__builtin_popcountll(m) << b;
    }
    if (total == 0) return false;
    ntri += c;
    bool ended = false;
    for (uint32_t base = 0; base < total; base += 64u) {
        if (want) {
            const uint32_t lo = pre > base ? pre : base;
            const uint32_t hi = min(pre + c, base + 64u);
            for (uint32_t q = lo; q < hi; q++) wl->owner[q - base] = lane;
        }
        wl->key[lane] = ~0ull;
        wave_lds_sync();
        const uint32_t pair = base + lane;
        const bool act = pair < total;
        const uint32_t o = act ? wl->owner[lane] : lane;
        Ray ro;
        ro.ox = lane_f(r.ox, o); ro.oy = lane_f(r.oy, o); ro.oz = lane_f(r.oz, o);
        ro.dx = lane_f(r.dx, o); ro.dy = lane_f(r.dy, o); ro.dz = lane_f(r.dz, o);
        ro.tmax = lane_f(r.tmax, o);
        const uint32_t k = lane_u(first, o) + (pair - lane_u(pre, o));
        bool hit = false;
        float t = 0.0f, u = 0.0f, v = 0.0f;
        uint32_t id = 0;
        if (act && k < ld.n_tris) {  // bounds guard; a valid tree never fails it
            if (LeafMode == BVH_LEAF_COMPACT) {
                const float4 *p = static_cast<const float4 *>(ld.leaf) + 3 * (size_t)k;
                const float4 a = p[0], b = p[1];
                const float2 cc = *reinterpret_cast<const float2 *>(p + 2);
                hit = mt_edges(ro, a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, cc.x, t, u, v);
                id = __float_as_uint(cc.y);
            } else {
                id = (uint32_t) static_cast<const int32_t *>(ld.leaf)[k];
                const int32_t *tv = ld.tris + 3 * (size_t)id;
                const float *a = ld.verts + 3 * (size_t)tv[0];
                const float *b = ld.verts + 3 * (size_t)tv[1];
                const float *cv = ld.verts + 3 * (size_t)tv[2];
                hit = mt(ro, a[0], a[1], a[2], b[0], b[1], b[2], cv[0], cv[1], cv[2], t, u, v);
            }
        }
        const unsigned long long mine = ((unsigned long long)__float_as_uint(t) << 32) | id;
        if (hit) atomicMin(&wl->key[o], mine);
        wave_lds_sync();
        if (hit && wl->key[o] == mine) wl->uv[o] = make_float2(u, v);
        wave_lds_sync();
        if (want) {
            const unsigned long long kb = wl->key[lane];
            if (kb != ~0ull) {
                const float2 q = wl->uv[lane];
                consider(best, __uint_as_float((uint32_t)(kb >> 32)), q.x, q.y, (uint32_t)kb);
                if (Mode == BVH_TRACE_ANY) ended = true;
            }
        }
        wave_lds_sync();
    }
    return ended;
}

// ---------------------------------------------------------------------------
// Traversal stacks.  An entry is a node reference (E = uint32_t, binary
// layouts) or a reference with its entry distance (E = uint64_t: the distance's
// bits in the upper word, so that entries compare like their distances, which
// are never negative).  A node visit makes room for its children once, then
// puts them: put() always writes the slot at the top and moves the top only
// when the entry is kept, so the put itself has no branch.  It therefore needs
// room for at least one entry even where it keeps none.
//   reset()       empties the stack
//   room(n)       n >= 1 entries fit (moving older ones away if need be);
//                 false: the ray is re-traced by the fallback pass
//   put(e, keep)  writes e at the top
//   take()        takes the top entry; kBottom when the stack is empty
// The top is kept in bytes of LDS, so that a slot's address is one VALU
// operation.
// ---------------------------------------------------------------------------
// kRefDone: no reference of a tree, and like a leaf's its low bit is 0, so
// that one bit tells whether a lane has an interior node to visit.
constexpr uint32_t kRefDone = 0xFFFFFFFEu;
// What an empty stack gives: no reference; with a distance, one that no bound
// culls (-inf).
template <typename E>
inline constexpr E kBottom = kRefEmpty;
template <>
inline constexpr uint64_t kBottom<uint64_t> = (uint64_t)0xFF800000u << 32 | kRefDone;

// Deep stack of one lane in global memory: kStackMax entries, the build's
// bound on what a ray can need.
template <typename E>
struct GlobalStack {
    uint64_t *ent;  // [kStackMax]
    uint32_t sp = 0;
    __device__ explicit GlobalStack(uint64_t *e) : ent(e) {}
    __device__ void reset() { sp = 0; }
    __device__ bool room(uint32_t) { return true; }
    __device__ void put(E e, bool keep) {
        if (keep && sp < (uint32_t)kStackMax) ent[sp++] = e;
    }
    __device__ E take() { return sp > 0 ? (E)ent[--sp] : kBottom<E>; }
};

// Stack of one lane of a persistent kernel: a ring of SL entries in LDS
// (one column per lane, so lanes never share a bank) over a spill area in
// global memory that belongs to the lane for the whole launch (a cap of 0
// leaves the ring alone).  No private (scratch) memory is used.  Where the ring lacks room, its oldest half
// (or all it holds, if less) moves to the spill area; when it is empty, a pop
// first brings the newest half of the spilled entries back.  Entries [0, lo) live in the spill area, entries
// [lo, sp) in the ring.  room() fails only when the spill area (cap entries)
// is full.  A lane's spill entries are contiguous, so moving half a ring
// writes or reads one run (a 64-byte line for SL = 16 and 8-byte entries)
// instead of SL scattered words.
struct SpillArea {
    uint64_t *ent;    // [waves of the launch][per_wave][cap] entries of at most 8 bytes
    uint32_t per_wave;  // lanes of a wave that may hold rays, the first ones (64 at most)
    uint32_t cap;     // spill entries per lane
};

template <typename E, int SL>
struct RingStack {
    static_assert((SL & (SL - 1)) == 0 && SL >= 2 && SL <= 32, "ring size must be a power of two");
    static constexpr uint32_t kStep = kTraceBlock * sizeof(E);
    static constexpr uint32_t kHalf = (SL / 2) * kStep;
    E *lds;               // [SL][kTraceBlock]
    SpillArea area;       // uniform across the launch
    uint32_t sp = 0, lo = 0;
    __device__ RingStack(E *l, const SpillArea &a) : lds(l), area(a) {}
    __device__ E &slot(uint32_t at) const {
        return *reinterpret_cast<E *>(reinterpret_cast<char *>(lds) +
                                      ((at & ((SL - 1) * kStep)) | (threadIdx.x * (uint32_t)sizeof(E))));
    }
    __device__ void reset() { sp = lo = 0; }
    __device__ uint32_t entries() const { return sp / kStep; }
    // all entries lie in the ring, from its first slot on, with room for one more
    __device__ bool in_ring() const { return lo == 0 && sp < SL * kStep; }
    // the lane's spill run, as entries of type E
    __device__ E *run() const {
        const size_t wave = (size_t)blockIdx.x * (kTraceBlock / 64) + (threadIdx.x >> 6);
        return reinterpret_cast<E *>(area.ent + (wave * area.per_wave + (threadIdx.x & 63u)) * area.cap);
    }
    __device__ bool room(uint32_t n) {
        while (sp - lo + n * kStep > SL * kStep) {
            const uint32_t m = min(kHalf, sp - lo);
            if (lo + m > area.cap * kStep) return false;
            E *to = run() + lo / kStep;
            for (uint32_t e = 0; e < m; e += kStep) to[e / kStep] = slot(lo + e);
            lo += m;
        }
        return true;
    }
    __device__ void put(E e, bool keep) {
        slot(sp) = e;
        sp += keep ? kStep : 0u;
    }
    __device__ E take() {
        if (sp == lo) refill();
        sp -= kStep;
        return slot(sp);
    }
    // the ring is empty: brings spilled entries back, or puts kBottom
    __device__ void refill() {
        if (lo == 0) {
            put(kBottom<E>, true);
            return;
        }
        const uint32_t m = min(kHalf, lo);
        lo -= m;
        const E *from = run() + lo / kStep;
        for (uint32_t e = 0; e < m; e += kStep) slot(lo + e) = from[e / kStep];
    }
};

__device__ inline void store_hit(bvh_hit *hits, uint64_t i, const Best &b) {
    int4 w;
    w.x = (b.id == 0xFFFFFFFFu) ? -1 : (int)b.id;
    w.y = __float_as_int(b.id == 0xFFFFFFFFu ? INFINITY : b.t);
    w.z = __float_as_int(b.id == 0xFFFFFFFFu ? 0.0f : b.u);
    w.w = __float_as_int(b.id == 0xFFFFFFFFu ? 0.0f : b.v);
    reinterpret_cast<int4 *>(hits)[i] = w;
}


// The distance that culls nodes: the best hit so far (closest-hit queries)
// or tmax, widened like the far distances of the slab test.
template <int Mode>
__device__ inline float cull_bound(const Ray &r, const Best &b) {
    return ((Mode == BVH_TRACE_ANY) ? r.tmax : fminf(b.t, r.tmax)) * kFarScale;
}

// ---------------------------------------------------------------------------
// Binary layout with the box in the node (AABB2): visit a node by testing its
// own box against the current best; a leaf's triangles are then tested, an
// interior node continues with the near child (split axis and ray direction
// sign) and pushes the far child.
// ---------------------------------------------------------------------------
struct BinState {
    Best best;
    float cull;     // boxes entered beyond this are culled: the best hit so far or tmax, widened
    uint32_t node;  // next node to visit; kRefEmpty when no node is left
    uint32_t leaf;  // leaf parked by the two-phase order (kRefEmpty: none)
    uint32_t hold;  // a second leaf met while one is parked; the lane then waits
    __device__ bool progress() const { return node != kRefEmpty && hold == kRefEmpty; }
};

__device__ inline BinState bin_start(int64_t n_nodes, const Ray &r) {
    BinState s;
    s.best = Best{INFINITY, 0.0f, 0.0f, 0xFFFFFFFFu};
    s.cull = r.tmax * kFarScale;
    s.node = n_nodes > 0 ? 0u : kRefEmpty;
    s.leaf = s.hold = kRefEmpty;
    return s;
}

// Binary node formats: load node i as its box, triangle count (0 for an
// interior node), offset (right-child delta or first triangle) and split
// axis (3 when unknown).
struct BinAABB2 {
    static constexpr bool kSplit = false;
    __device__ static void load(const void *nodes, uint32_t i, const SceneData &, float *lo,
                                float *hi, uint32_t &cnt, uint32_t &off, uint32_t &axis) {
        const float4 *np = reinterpret_cast<const float4 *>(static_cast<const bvh_node_aabb2 *>(nodes) + i);
        const float4 a = np[0], b = np[1];
        lo[0] = a.x; lo[1] = a.y; lo[2] = a.z;
        hi[0] = a.w; hi[1] = b.x; hi[2] = b.y;
        off = __float_as_uint(b.z);
        const uint32_t meta = __float_as_uint(b.w);
        cnt = meta & 0xFFFFu;
        axis = (meta >> 16) & 3u;
    }
};

// pbrt-q16: one 16-B load; planes dequantised in the scene frame.
struct BinPbrtQ16 {
    static constexpr bool kSplit = false;
    __device__ static void load(const void *nodes, uint32_t i, const SceneData &sd, float *lo,
                                float *hi, uint32_t &cnt, uint32_t &off, uint32_t &axis) {
        const uint4 w = reinterpret_cast<const uint4 *>(nodes)[i];
        const uint32_t q[6] = {w.x & 0xFFFFu, w.x >> 16, w.y & 0xFFFFu,
                               w.y >> 16,     w.z & 0xFFFFu, w.z >> 16};
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fmaf((float)q[a], sd.fs[a], sd.fo[a]);
            hi[a] = fmaf((float)q[3 + a], sd.fs[a], sd.fo[a]);
        }
        cnt = w.w & 0xFu;
        off = w.w >> 4;
        axis = (q[0] & 1u) | ((q[1] & 1u) << 1);
    }
};

// sg-eq: one 12-B load; 10-bit planes counted up from the frame origin
// (lower) and down from the frame top (upper).
struct BinSgEq {
    static constexpr bool kSplit = false;
    __device__ static void load(const void *nodes, uint32_t i, const SceneData &sd, float *lo,
                                float *hi, uint32_t &cnt, uint32_t &off, uint32_t &axis) {
        const uint32_t *p = static_cast<const uint32_t *>(nodes) + 3 * (size_t)i;
        const uint32_t ql = p[0], qh = p[1], w = p[2];
        const uint32_t qlo[3] = {(ql >> 20) & 1023u, (ql >> 10) & 1023u, ql & 1023u};
        const uint32_t qhi[3] = {(qh >> 20) & 1023u, (qh >> 10) & 1023u, qh & 1023u};
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fmaf((float)qlo[a], sd.fs[a], sd.fo[a]);
            hi[a] = fmaf(-(float)qhi[a], sd.fs[a], sd.ft[a]);
        }
        cnt = (ql >> 30) | ((qh >> 30) << 2);
        off = w & 0x3FFFFFFFu;
        axis = cnt > 0 ? 3u : (w >> 30);
    }
};

// Split layouts (box array, then topology array): load_box fetches only the
// box, load_meta the topology word(s), so a node whose box the query misses
// costs one fetch; load fetches both.
struct BinPbrtSoAoS {
    static constexpr bool kSplit = true;
    __device__ static void load_box(const void *nodes, uint32_t i, const SceneData &, float *lo,
                                    float *hi) {
        const float2 *p = static_cast<const float2 *>(nodes) + 3 * (size_t)i;
        const float2 a = p[0], b = p[1], c = p[2];
        lo[0] = a.x; lo[1] = a.y; lo[2] = b.x;
        hi[0] = b.y; hi[1] = c.x; hi[2] = c.y;
    }
    __device__ static void load_meta(uint32_t i, const SceneData &sd, uint32_t &cnt, uint32_t &off,
                                     uint32_t &axis) {
        const uint2 t = static_cast<const uint2 *>(sd.topo)[i];
        off = t.x;
        cnt = t.y & 0xFFFFu;
        axis = (t.y >> 16) & 3u;
    }
    __device__ static void load(const void *nodes, uint32_t i, const SceneData &sd, float *lo,
                                float *hi, uint32_t &cnt, uint32_t &off, uint32_t &axis) {
        load_box(nodes, i, sd, lo, hi);
        load_meta(i, sd, cnt, off, axis);
    }
};

struct BinPbrtQ16SoAoS {
    static constexpr bool kSplit = true;
    // boxes are 12 B: entry i starts at word 3 i (u16 pairs lo_x|lo_y, lo_z|hi_x, hi_y|hi_z)
    __device__ static void load_box_q(const void *nodes, uint32_t i, uint32_t *q) {
        const uint32_t *p = static_cast<const uint32_t *>(nodes) + 3 * (size_t)i;
        const uint32_t w0 = p[0], w1 = p[1], w2 = p[2];
        q[0] = w0 & 0xFFFFu; q[1] = w0 >> 16; q[2] = w1 & 0xFFFFu;
        q[3] = w1 >> 16;     q[4] = w2 & 0xFFFFu; q[5] = w2 >> 16;
    }
    __device__ static void load_box(const void *nodes, uint32_t i, const SceneData &sd, float *lo,
                                    float *hi) {
        uint32_t q[6];
        load_box_q(nodes, i, q);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fmaf((float)q[a], sd.fs[a], sd.fo[a]);
            hi[a] = fmaf((float)q[3 + a], sd.fs[a], sd.fo[a]);
        }
    }
    // the split axis lives in the box (lowest bits of lo_x and lo_y)
    __device__ static void load_meta_axis(const void *nodes, uint32_t i, const SceneData &sd,
                                          uint32_t &cnt, uint32_t &off, uint32_t &axis) {
        const uint32_t m = static_cast<const uint32_t *>(sd.topo)[i];
        cnt = m & 0xFu;
        off = m >> 4;
        const uint32_t w0 = static_cast<const uint32_t *>(nodes)[3 * (size_t)i];
        axis = (w0 & 1u) | ((w0 >> 16) & 1u) << 1;
    }
    __device__ static void load(const void *nodes, uint32_t i, const SceneData &sd, float *lo,
                                float *hi, uint32_t &cnt, uint32_t &off, uint32_t &axis) {
        uint32_t q[6];
        load_box_q(nodes, i, q);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fmaf((float)q[a], sd.fs[a], sd.fo[a]);
            hi[a] = fmaf((float)q[3 + a], sd.fs[a], sd.fo[a]);
        }
        const uint32_t m = static_cast<const uint32_t *>(sd.topo)[i];
        cnt = m & 0xFu;
        off = m >> 4;
        axis = (q[0] & 1u) | ((q[1] & 1u) << 1);
    }
};

// sg-eq records padded to 16 B: one aligned 16-byte fetch.
struct BinSgEqA16 {
    static constexpr bool kSplit = false;
    __device__ static void load(const void *nodes, uint32_t i, const SceneData &sd, float *lo,
                                float *hi, uint32_t &cnt, uint32_t &off, uint32_t &axis) {
        const uint4 r = static_cast<const uint4 *>(nodes)[i];
        const uint32_t ql = r.x, qh = r.y, w = r.z;
        const uint32_t qlo[3] = {(ql >> 20) & 1023u, (ql >> 10) & 1023u, ql & 1023u};
        const uint32_t qhi[3] = {(qh >> 20) & 1023u, (qh >> 10) & 1023u, qh & 1023u};
#pragma unroll
        for (int a = 0; a < 3; a++) {
            lo[a] = fmaf((float)qlo[a], sd.fs[a], sd.fo[a]);
            hi[a] = fmaf(-(float)qhi[a], sd.fs[a], sd.ft[a]);
        }
        cnt = (ql >> 30) | ((qh >> 30) << 2);
        off = w & 0x3FFFFFFFu;
        axis = cnt > 0 ? 3u : (w >> 30);
    }
};

// Split-layout meta fetch (the pbrt-q16 variant re-reads the box's first word
// for the axis bits, a cache hit after the box fetch).
template <class Node>
__device__ inline void split_meta(const void *nodes, uint32_t i, const SceneData &sd, uint32_t &cnt,
                                  uint32_t &off, uint32_t &axis) {
    if constexpr (std::is_same_v<Node, BinPbrtQ16SoAoS>)
        Node::load_meta_axis(nodes, i, sd, cnt, off, axis);
    else
        Node::load_meta(i, sd, cnt, off, axis);
}

// Whether a round's interior phase ends, with lanes `prog` that can go on and
// `parked` that have a leaf to test.  A coherent wave leaves at most
// kCoherentStall lanes behind that have no leaf yet.  Camera rays on a terrain
// of 382,000 triangles, 1 M without allocation, at 0 / 4 / 8 / 16: 10-bit binary
// nodes 450 / 398 / 383 / 382 us, AABB2 330 / 305 / 296 / 297, BVH8-Q8 185 / 178 /
// 177 / 177.  BVH4 waits for every lane: 157 / 155 / 155 / 157, but 2 M in a
// persistent launch 290 / 295 / 298 / 304.
template <uint32_t kCoherentStall, uint32_t kStall>
__device__ inline bool phase_over(bool coherent, uint64_t prog, uint64_t parked) {
    if (coherent) {
        const uint32_t late = (uint32_t)__builtin_popcountll(prog & ~parked);
        return late == 0 || (kCoherentStall > 0 && late <= kCoherentStall && parked != 0);
    }
    return prog == 0 || ((uint32_t)__builtin_popcountll(prog) <= kStall && parked != 0);
}

// Visits bs.node: an interior node whose box the ray meets continues with the
// near child (split axis and ray direction sign) and stacks the far one; a
// leaf whose box it meets is parked (or held, if one is parked already).
// bs.node moves on to the next node.  The node's loads are issued at a raised
// priority, as in the wide layouts' visits.
template <class Node, class Stack>
__device__ inline void bin_visit(const void *nodes, int64_t n_nodes, const SceneData &sd,
                                 const Ray &r, bool fast, Stack &st, BinState &bs,
                                 uint32_t &nfetch, bool &incomplete) {
    // bounds guard; equal on a valid tree
    const uint32_t at = min(bs.node, (uint32_t)n_nodes - 1u);
    float lo[3], hi[3];
    uint32_t cnt = 0, off = 0, axis = 0;
    __builtin_amdgcn_s_setprio(3);
    if constexpr (Node::kSplit)
        Node::load_box(nodes, at, sd, lo, hi);
    else
        Node::load(nodes, at, sd, lo, hi, cnt, off, axis);
    __builtin_amdgcn_s_setprio(0);
    nfetch++;
    const float tn = fast ? slab<true>(r, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], bs.cull)
                          : slab<false>(r, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], bs.cull);
    const bool met = tn != INFINITY;
    if constexpr (Node::kSplit)
        if (met) split_meta<Node>(nodes, at, sd, cnt, off, axis);
    if (met && cnt == 0) {
        const bool neg = axis == 0 ? r.nx : (axis == 1 ? r.ny : (axis == 2 ? r.nz : false));
        const uint32_t left = at + 1, right = at + off;
        if (st.room(1)) {
            st.put(neg ? left : right, true);
            bs.node = neg ? right : left;
        } else {
            incomplete = true;
            bs.node = bs.leaf = bs.hold = kRefEmpty;
        }
        return;
    }
    if (met) {
        const uint32_t leaf = ref_leaf(off, cnt);
        if (bs.leaf == kRefEmpty) bs.leaf = leaf;
        else bs.hold = leaf;
    }
    bs.node = st.take();
}

// After the parked leaf has been tested; a satisfied any-hit query ends the
// ray.
template <int Mode>
__device__ inline void bin_tested(const Ray &r, bool ended, BinState &bs) {
    bs.leaf = bs.hold;
    bs.hold = kRefEmpty;
    if (ended) bs.node = bs.leaf = kRefEmpty;
    if (Mode == BVH_TRACE_CLOSEST) bs.cull = cull_bound<Mode>(r, bs.best);
}

// Tests the parked leaf in the lane.
template <int LeafMode, int Mode>
__device__ inline void bin_test_parked(const SceneData &ld, const Ray &r, BinState &bs,
                                       uint32_t &ntri) {
    const uint32_t first = bs.leaf >> 5, cnt = ((bs.leaf >> 1) & 0xFu) + 1u;
    bin_tested<Mode>(r, test_leaf<LeafMode, Mode>(ld, r, first, cnt, bs.best, ntri), bs);
}

// ---------------------------------------------------------------------------
// Wide layouts: the node holds its children's boxes.  Decoders expose
//   K                      arity
//   kWords                 16-byte words of a node that a visit reads
//   Prep prep(ray)         per-ray constants
//   fetch(node buffer, node, prep, m)   those words, m[kWords]
//   test(m, ray, cull, tn[K], ref[K])
// test writes the entry distance of every child the ray meets (+inf
// otherwise).  Node buffers of the wide layouts are below 4 GiB (the builder
// sees to it), so each load is base + one 32-bit offset.
//
// What bounds a visit of scattered rays is the vector L1: it serves one lookup per
// clock (a wave's load of 16 bytes per lane from 64 lines takes 65 clocks,
// measured), so a visit's seven loads occupy it for 448, and the 64 lines of
// each of the CU's 16 waves together exceed its 32 KB: a line that leaves
// between two loads of one wave is fetched again.  The wave's priority is
// therefore raised while it issues a visit's loads, so that the waves of a
// SIMD do not take turns at theirs (BVH4: bounce rays of the terrain 572 -> 507 us, 4 M
// uniform rays on the spheres scene 11.1 -> 9.4 ms).
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__host__ __device__ inline float as_f32(uint32_t x) { return __builtin_bit_cast(float, x); }
struct NoPrep {};

// BVH4: the near and far plane arrays of an axis are picked by address (the
// sign of the direction component decides whether lo_a or hi_a is entered
// first), so the per-child slab test needs no plane selects.
struct DecodeBVH4 {
    static constexpr int K = 4;
    static constexpr int kWords = 7;
    // scattered waves end a round's interior phase at <= kStall progressing
    // lanes (terrain bounce rays: 0.616 / 0.600 / 0.577 / 0.559 / 0.563 /
    // 0.585 / 0.646 ms at 8 / 16 / 24 / 32 / 40 / 48 / 56)
    static constexpr uint32_t kStall = 32;
    static constexpr uint32_t kCoherentStall = 0;  // see phase_over
    struct Prep {
        uint32_t nx, ny, nz;  // byte offsets of the entry-plane arrays in a node
    };
    __host__ __device__ static Prep prep(const Ray &r) {
        Prep p;
        p.nx = r.nx ? 48u : 0u;
        p.ny = r.ny ? 64u : 16u;
        p.nz = r.nz ? 80u : 32u;
        return p;
    }
    // m: entry planes of x, y, z, exit planes of x, y, z, references.  The
    // offsets of the two plane arrays of an axis (0 and 48, 16 and 64, 32 and
    // 80) turn into each other by one exclusive or, also in 128-byte aligned
    // nodes' addresses.
    __host__ __device__ static void fetch(const void *nodes, uint32_t node, const Prep &p, u32x4 *m) {
        const char *b = static_cast<const char *>(nodes);
        const uint32_t o = node << 7, x = o + p.nx, y = o + p.ny, z = o + p.nz;
        m[0] = *reinterpret_cast<const u32x4 *>(b + x);
        m[1] = *reinterpret_cast<const u32x4 *>(b + y);
        m[2] = *reinterpret_cast<const u32x4 *>(b + z);
        m[3] = *reinterpret_cast<const u32x4 *>(b + (x ^ 48u));
        m[4] = *reinterpret_cast<const u32x4 *>(b + (y ^ 80u));
        m[5] = *reinterpret_cast<const u32x4 *>(b + (z ^ 112u));
        m[6] = *reinterpret_cast<const u32x4 *>(b + (size_t)o + 96);
    }
    template <bool Fast>
    __host__ __device__ static void test(const u32x4 *m, const Ray &r, float cull, float *tn,
                                         uint32_t *ref) {
#pragma unroll
        for (int c = 0; c < 4; c++) {
            tn[c] = slab_nf<Fast>(r, as_f32(m[0][c]), as_f32(m[1][c]), as_f32(m[2][c]),
                                  as_f32(m[3][c]), as_f32(m[4][c]), as_f32(m[5][c]), cull);
            ref[c] = m[6][c];
            // an empty slot's infinite planes cull it, unless every distance is NaN
            // (not with Fast, whose 1/d is finite and not zero)
            if (!Fast && ref[c] == kRefEmpty) tn[c] = INFINITY;
        }
    }
};

// Byte c of the 8 packed bytes held in words (w0, w1).
__host__ __device__ inline uint32_t byte_of(uint32_t w0, uint32_t w1, int c) {
    return ((c < 4 ? w0 : w1) >> (8 * (c & 3))) & 0xFFu;
}
__host__ __device__ inline uint32_t half_of(const uint32_t *w, int c) {
    return (w[c >> 1] >> (16 * (c & 1))) & 0xFFFFu;
}

// Quantised layouts: the near/far choice is made once per packed word (four
// u8 or two u16 planes at a time) before dequantising.
template <int NodeBytes, int Words>
struct DecodeBVH8 {
    static constexpr int K = 8;
    static constexpr int kWords = Words;
    // as DecodeBVH4::kStall (terrain bounce rays, BVH8-Q8: 0.705 / 0.653 /
    // 0.620 / 0.632 / 0.665 ms at 16 / 32 / 40 / 48 / 56)
    static constexpr uint32_t kStall = 40;
    static constexpr uint32_t kCoherentStall = 8;
    using Prep = NoPrep;
    __host__ __device__ static Prep prep(const Ray &) { return Prep{}; }
    __host__ __device__ static void fetch(const void *nodes, uint32_t node, const Prep &, u32x4 *m) {
        const char *b = static_cast<const char *>(nodes) + (size_t)(node * (uint32_t)NodeBytes);
#pragma unroll
        for (int k = 0; k < Words; k++) m[k] = reinterpret_cast<const u32x4 *>(b)[k];
    }
};

struct DecodeBVH8Q8 : DecodeBVH8<sizeof(bvh_node_bvh8_q8), 7> {
    template <bool Fast>
    __host__ __device__ static void test(const u32x4 *m, const Ray &r, float cull, float *tn,
                                         uint32_t *ref) {
        uint32_t w[28];
#pragma unroll
        for (int k = 0; k < 28; k++) w[k] = m[k / 4][k % 4];
        const float ox = as_f32(w[0]), oy = as_f32(w[1]), oz = as_f32(w[2]);
        const float sx = as_f32(w[3]), sy = as_f32(w[4]), sz = as_f32(w[5]);
        // words: lo_x 6-7, lo_y 8-9, lo_z 10-11, hi_x 12-13, hi_y 14-15, hi_z 16-17
        uint32_t n[6], f[6];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            n[k] = r.nx ? w[12 + k] : w[6 + k];
            f[k] = r.nx ? w[6 + k] : w[12 + k];
            n[2 + k] = r.ny ? w[14 + k] : w[8 + k];
            f[2 + k] = r.ny ? w[8 + k] : w[14 + k];
            n[4 + k] = r.nz ? w[16 + k] : w[10 + k];
            f[4 + k] = r.nz ? w[10 + k] : w[16 + k];
        }
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const float nxp = fmaf((float)byte_of(n[0], n[1], c), sx, ox);
            const float nyp = fmaf((float)byte_of(n[2], n[3], c), sy, oy);
            const float nzp = fmaf((float)byte_of(n[4], n[5], c), sz, oz);
            const float fxp = fmaf((float)byte_of(f[0], f[1], c), sx, ox);
            const float fyp = fmaf((float)byte_of(f[2], f[3], c), sy, oy);
            const float fzp = fmaf((float)byte_of(f[4], f[5], c), sz, oz);
            const bool valid = (uint32_t)c < w[26];
            tn[c] = valid ? slab_nf<Fast>(r, nxp, nyp, nzp, fxp, fyp, fzp, cull) : INFINITY;
            ref[c] = w[18 + c];
        }
    }
};

struct DecodeBVH8Q16 : DecodeBVH8<sizeof(bvh_node_bvh8_q16), 10> {
    template <bool Fast>
    __host__ __device__ static void test(const u32x4 *m, const Ray &r, float cull, float *tn,
                                         uint32_t *ref) {
        uint32_t w[40];
#pragma unroll
        for (int k = 0; k < 40; k++) w[k] = m[k / 4][k % 4];
        const float ox = as_f32(w[0]), oy = as_f32(w[1]), oz = as_f32(w[2]);
        const float sx = as_f32(w[3]), sy = as_f32(w[4]), sz = as_f32(w[5]);
        // words: lo_x 6-9, lo_y 10-13, lo_z 14-17, hi_x 18-21, hi_y 22-25, hi_z 26-29
        uint32_t n[12], f[12];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            n[k] = r.nx ? w[18 + k] : w[6 + k];
            f[k] = r.nx ? w[6 + k] : w[18 + k];
            n[4 + k] = r.ny ? w[22 + k] : w[10 + k];
            f[4 + k] = r.ny ? w[10 + k] : w[22 + k];
            n[8 + k] = r.nz ? w[26 + k] : w[14 + k];
            f[8 + k] = r.nz ? w[14 + k] : w[26 + k];
        }
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const float nxp = fmaf((float)half_of(n, c), sx, ox);
            const float nyp = fmaf((float)half_of(n + 4, c), sy, oy);
            const float nzp = fmaf((float)half_of(n + 8, c), sz, oz);
            const float fxp = fmaf((float)half_of(f, c), sx, ox);
            const float fyp = fmaf((float)half_of(f + 4, c), sy, oy);
            const float fzp = fmaf((float)half_of(f + 8, c), sz, oz);
            const bool valid = (uint32_t)c < w[38];
            tn[c] = valid ? slab_nf<Fast>(r, nxp, nyp, nzp, fxp, fyp, fzp, cull) : INFINITY;
            ref[c] = w[30 + c];
        }
    }
};

// A stack entry of a wide traversal: entry distance (never negative) above
// the reference.
__device__ inline uint64_t entry_of(float t, uint32_t ref) {
    return ((uint64_t)__float_as_uint(t) << 32) | ref;
}
__device__ inline float entry_t(uint64_t e) { return __uint_as_float((uint32_t)(e >> 32)); }
__device__ inline uint32_t entry_ref(uint64_t e) { return (uint32_t)e; }

// Orders two entries.  Read as 64-bit floats they are positive and finite
// (the f32 infinity's bits in the upper word are a finite f64), so the f64
// minimum and maximum order them as integers would, in two full-rate VALU
// instructions (measured 5.8 cycles each per wave, v_min_f32 5.6) where a
// compare and selects take five.  Denormals are kept in f64.
__device__ inline void order_entries(uint64_t &a, uint64_t &b) {
    const double x = __longlong_as_double((long long)a), y = __longlong_as_double((long long)b);
    double lo, hi;
    asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(x), "v"(y));
    asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(x), "v"(y));
    a = (uint64_t)__double_as_longlong(lo);
    b = (uint64_t)__double_as_longlong(hi);
}

// Ascending sort by entry distance (sorting networks: 5 and 19 exchanges).
template <int K>
__device__ inline void sort_entries(uint64_t *e) {
    if (K == 4) {
        order_entries(e[0], e[1]); order_entries(e[2], e[3]);
        order_entries(e[0], e[2]); order_entries(e[1], e[3]);
        order_entries(e[1], e[2]);
    } else {
        order_entries(e[0], e[2]); order_entries(e[1], e[3]);
        order_entries(e[4], e[6]); order_entries(e[5], e[7]);
        order_entries(e[0], e[4]); order_entries(e[1], e[5]);
        order_entries(e[2], e[6]); order_entries(e[3], e[7]);
        order_entries(e[0], e[1]); order_entries(e[2], e[3]);
        order_entries(e[4], e[5]); order_entries(e[6], e[7]);
        order_entries(e[2], e[4]); order_entries(e[3], e[5]);
        order_entries(e[1], e[4]); order_entries(e[3], e[6]);
        order_entries(e[1], e[2]); order_entries(e[3], e[4]); order_entries(e[5], e[6]);
    }
}

// Puts the kept ones of the sorted entries e[1..K) on the stack, farthest
// first (the kept ones come before the others, whose distance is +inf).
// False when the stack has no room for them.
template <int K, class Stack>
__device__ inline bool put_rest(Stack &st, const uint64_t *e) {
    uint32_t n = 0;
#pragma unroll
    for (int c = 1; c < K; c++) n += entry_t(e[c]) != INFINITY ? 1u : 0u;
    if (!st.room(n > 0 ? n : 1u)) return false;
#pragma unroll
    for (int c = K - 1; c >= 1; c--) st.put(e[c], entry_t(e[c]) != INFINITY);
    return true;
}

// Traversal state of one ray in a wide BVH.
struct WideState {
    Best best;
    float cull;      // boxes entered beyond this are culled: the best hit so far or tmax, widened
    uint64_t cur;    // entry to visit next; reference kRefDone once the ray is done
    uint32_t leaf;   // leaf parked by the two-phase order (kRefDone: none)
    __device__ bool interior() const { return ((uint32_t)cur & 1u) != 0u; }
    __device__ bool live() const { return entry_ref(cur) != kRefDone; }
    // parks the leaf at hand if none is parked; true: the lane needs another entry
    __device__ bool park() {
        const bool p = !interior() && live() && leaf == kRefDone;
        leaf = p ? entry_ref(cur) : leaf;
        return p;
    }
};

__device__ inline WideState wide_start(int64_t n_nodes, const Ray &r) {
    WideState ws;
    ws.best = Best{INFINITY, 0.0f, 0.0f, 0xFFFFFFFFu};
    ws.cull = fminf(r.tmax, INFINITY) * kFarScale;  // a NaN tmax culls no box (and accepts no hit)
    ws.cur = entry_of(0.0f, n_nodes > 0 && ray_finite(r) ? ref_interior(0) : kRefDone);
    ws.leaf = kRefDone;
    return ws;
}

// A closest-hit ray's culling distance after its best hit may have changed.
template <int Mode>
__device__ inline void wide_update_cull(const Ray &r, WideState &ws) {
    if (Mode == BVH_TRACE_CLOSEST) ws.cull = cull_bound<Mode>(r, ws.best);
}

// One advance of a lane: visits the interior node at hand (tests all its
// children, sorts those the ray meets near-first, stacks all but the nearest
// with their entry distances and continues with the nearest); a leaf reached
// this way or from the stack is parked if none is parked yet, and the lane
// takes its next unculled entry from the stack.  Afterwards ws.cur is an
// interior node, a leaf while another is parked, or kRefDone.  A stack
// without room ends the ray as incomplete.
template <class Dec, int Mode, class Stack>
__device__ inline void wide_advance(const void *nodes, uint32_t last, const Ray &r,
                                    const typename Dec::Prep &prep, bool fast, Stack &st,
                                    WideState &ws, uint32_t &nfetch, bool &incomplete) {
    constexpr int K = Dec::K;
    bool pop = false;
    if (ws.interior()) {
        float tn[K];
        uint32_t ref[K];
        u32x4 m[Dec::kWords];
        __builtin_amdgcn_s_setprio(3);
        // the index is clamped as a bounds guard, which a valid tree never needs
        Dec::fetch(nodes, min((uint32_t)ws.cur >> 1, last), prep, m);
        __builtin_amdgcn_s_setprio(0);
        if (fast)
            Dec::template test<true>(m, r, ws.cull, tn, ref);
        else
            Dec::template test<false>(m, r, ws.cull, tn, ref);
        nfetch++;
        uint64_t e[K];
#pragma unroll
        for (int c = 0; c < K; c++) e[c] = entry_of(tn[c], ref[c]);
        sort_entries<K>(e);
        ws.cur = e[0];
        pop = entry_t(e[0]) == INFINITY;
        if (!put_rest<K>(st, e)) {
            incomplete = true;
            st.reset();
            pop = true;
        }
    }
    if (!pop) pop = ws.park();
    while (pop) {
        const uint64_t e = st.take();
        const bool keep = entry_t(e) <= ws.cull;
        ws.cur = keep ? e : ws.cur;
        pop = !keep || ws.park();
    }
}

// Takes the next unculled entry where the one at hand was taken before the
// best hit improved and is culled by now.
template <class Stack>
__device__ inline void wide_recull(Stack &st, WideState &ws) {
    while (!(entry_t(ws.cur) <= ws.cull)) ws.cur = st.take();
}

// Tests the triangles of the parked leaf in the lane; a satisfied any-hit
// query ends the ray.
template <int LeafMode, int Mode, class Stack>
__device__ inline void wide_test_parked(const SceneData &ld, const Ray &r, Stack &st, WideState &ws,
                                        uint32_t &ntri) {
    const uint32_t first = ws.leaf >> 5, cnt = ((ws.leaf >> 1) & 0xFu) + 1u;
    ws.leaf = kRefDone;
    if (test_leaf<LeafMode, Mode>(ld, r, first, cnt, ws.best, ntri)) {
        ws.cur = kBottom<uint64_t>;
        return;
    }
    wide_update_cull<Mode>(r, ws);
    wide_recull(st, ws);
}

// Visits one stack entry by itself: an interior node's children that the ray
// meets, near-first, in kids[0..n), or a leaf's reference.
template <class Dec>
__device__ inline void wide_expand(const void *nodes, uint32_t last, const Ray &r,
                                   const typename Dec::Prep &prep, bool fast, float cull,
                                   uint64_t entry, uint64_t *kids, uint32_t &n, uint32_t &leaf) {
    if (!(entry_t(entry) <= cull)) return;
    if (!(entry_ref(entry) & 1u)) {
        leaf = entry_ref(entry);
        return;
    }
    constexpr int K = Dec::K;
    float tn[K];
    uint32_t ref[K];
    u32x4 m[Dec::kWords];
    Dec::fetch(nodes, min(entry_ref(entry) >> 1, last), prep, m);
    if (fast)
        Dec::template test<true>(m, r, cull, tn, ref);
    else
        Dec::template test<false>(m, r, cull, tn, ref);
#pragma unroll
    for (int c = 0; c < K; c++) {
        kids[c] = entry_of(tn[c], ref[c]);
        n += tn[c] != INFINITY ? 1u : 0u;
    }
    sort_entries<K>(kids);
}

// One round of the two-phase order (the while-while scheme of Aila and Laine
// 2009, with speculative traversal), called by every lane of the wave (lanes
// without a ray hold kRefDone), so that the lanes test nodes together and
// triangles together instead of splitting every step between the two:
//   interior phase: lanes visit interior nodes, park the first leaf they
//     meet and keep descending; a lane whose next entry is a second leaf
//     waits.  With coherent rays the phase ends when all lanes but a few have
//     a parked leaf or are done; with scattered rays once at most kStall lanes
//     can still make progress (waiting for the last stragglers of such a wave
//     would idle the rest);
//   leaf phase: the parked leaves are tested, each in its lane where the
//     rays are coherent (their lanes hold leaves at the same time), else in
//     one wave-batched leaf phase.
// Every node that the current best does not cull is still visited, so the
// result equals the plain order's.
template <class Dec, int LeafMode, int Mode, class Stack>
__device__ inline void wide_round(const void *nodes, uint32_t last, const SceneData &ld,
                                  const Ray &r, const typename Dec::Prep &prep, bool fast,
                                  bool coherent, Stack &st, WideState &ws, WaveLeafLds *wl,
                                  uint32_t &nfetch, uint32_t &ntri, bool &incomplete) {
    for (;;) {
        wide_advance<Dec, Mode>(nodes, last, r, prep, fast, st, ws, nfetch, incomplete);
        const uint64_t prog = __builtin_amdgcn_ballot_w64(ws.interior());
        const uint64_t parked = __builtin_amdgcn_ballot_w64(ws.leaf != kRefDone);
        if (phase_over<Dec::kCoherentStall, Dec::kStall>(coherent, prog, parked)) break;
    }
    if (coherent) {
        if (ws.leaf != kRefDone) wide_test_parked<LeafMode, Mode>(ld, r, st, ws, ntri);
        return;
    }
    const bool want = ws.leaf != kRefDone;
    const uint32_t first = ws.leaf >> 5, cnt = ((ws.leaf >> 1) & 0xFu) + 1u;
    const bool ended = wave_test_leaves<LeafMode, Mode>(ld, r, want, first, cnt, ws.best, ntri, wl);
    if (want) {
        ws.leaf = kRefDone;
        wide_update_cull<Mode>(r, ws);
        if (ended) ws.cur = kBottom<uint64_t>;
        wide_recull(st, ws);
    }
}

// ---------------------------------------------------------------------------
// Tracer policies: the per-layout state and steps behind one interface, so
// the kernels (one ray per lane, persistent, fallback, batched) are written
// once for all layouts.
//   Entry               stack entry (a reference, or one with its distance)
//   Prep prep(ray)      per-ray layout constants
//   State start(nodes, ray), none()   a ray's initial state, that of no ray
//   done(state); parked(state): a leaf waits to be tested; next(state): the
//                       entry a ray under way visits next
//   kChildren, expand(...)      the children of one stack entry, or its leaf
//   step<LeafMode, Mode>(...)   one advance of a lane on its own, and its leaf
//   wave<LeafMode, Mode>(...)   one round of the wave: every lane calls it,
//                               lanes without a ray with the state none()
// ---------------------------------------------------------------------------
template <class Dec>
struct WideTracer {
    using Entry = uint64_t;
    using State = WideState;
    using Prep = typename Dec::Prep;
    __device__ static Prep prep(const Ray &r) { return Dec::prep(r); }
    __device__ static State start(int64_t n_nodes, const Ray &r) { return wide_start(n_nodes, r); }
    __device__ static State none() { return wide_start(0, Ray{}); }
    __device__ static bool done(const State &s) { return !s.live() && s.leaf == kRefDone; }
    __device__ static bool parked(const State &s) { return s.leaf != kRefDone; }
    __device__ static Entry next(const State &s) { return s.cur; }
    static constexpr int kChildren = Dec::K;
    __device__ static void expand(const void *nodes, int64_t n_nodes, const SceneData &,
                                  const Ray &r, const Prep &prep, bool fast, float cull, Entry e,
                                  Entry *kids, uint32_t &n, uint32_t &leaf) {
        wide_expand<Dec>(nodes, (uint32_t)n_nodes - 1u, r, prep, fast, cull, e, kids, n, leaf);
    }
    template <int LeafMode, int Mode, class Stack>
    __device__ static void step(const void *nodes, int64_t n_nodes, const SceneData &ld,
                                const Ray &r, const Prep &prep, bool fast, Stack &st, State &s,
                                uint32_t &nfetch, uint32_t &ntri, bool &incomplete) {
        wide_advance<Dec, Mode>(nodes, (uint32_t)n_nodes - 1u, r, prep, fast, st, s, nfetch,
                                incomplete);
        if (s.leaf != kRefDone) wide_test_parked<LeafMode, Mode>(ld, r, st, s, ntri);
    }
    template <int LeafMode, int Mode, class Stack>
    __device__ static void wave(const void *nodes, int64_t n_nodes, const SceneData &ld,
                                const Ray &r, const Prep &prep, bool fast, bool coherent, Stack &st,
                                State &s, WaveLeafLds *wl, uint32_t &nfetch, uint32_t &ntri,
                                bool &incomplete) {
        wide_round<Dec, LeafMode, Mode>(nodes, (uint32_t)n_nodes - 1u, ld, r, prep, fast, coherent,
                                        st, s, wl, nfetch, ntri, incomplete);
    }
};

template <class Node>
struct BinTracer {
    using Entry = uint32_t;
    using State = BinState;
    using Prep = NoPrep;
    // as DecodeBVH4::kStall (AABB2, terrain bounce rays: 1.82 ms visiting one
    // node per step and testing leaves in their lanes; 1.24 / 1.10 / 1.07 ms
    // with this round at 16 / 32 / 48)
    static constexpr uint32_t kStall = 40;
    static constexpr uint32_t kCoherentStall = 8;
    __device__ static Prep prep(const Ray &) { return Prep{}; }
    __device__ static State start(int64_t n_nodes, const Ray &r) { return bin_start(n_nodes, r); }
    __device__ static State none() { return bin_start(0, Ray{}); }
    __device__ static bool done(const State &s) { return s.node == kRefEmpty && s.leaf == kRefEmpty; }
    __device__ static bool parked(const State &s) { return s.leaf != kRefEmpty; }
    __device__ static Entry next(const State &s) { return s.node; }
    static constexpr int kChildren = 2;
    __device__ static void expand(const void *nodes, int64_t n_nodes, const SceneData &ld,
                                  const Ray &r, const Prep &, bool fast, float cull, Entry e,
                                  Entry *kids, uint32_t &n, uint32_t &leaf) {
        const uint32_t at = min(e, (uint32_t)n_nodes - 1u);  // bounds guard; equal on a valid tree
        float lo[3], hi[3];
        uint32_t cnt = 0, off = 0, axis = 0;
        Node::load(nodes, at, ld, lo, hi, cnt, off, axis);
        const float tn = fast ? slab<true>(r, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], cull)
                              : slab<false>(r, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], cull);
        if (tn == INFINITY) return;
        if (cnt > 0) {
            leaf = ref_leaf(off, cnt);
            return;
        }
        const bool neg = axis == 0 ? r.nx : (axis == 1 ? r.ny : (axis == 2 ? r.nz : false));
        kids[0] = neg ? at + off : at + 1u;
        kids[1] = neg ? at + 1u : at + off;
        n = 2;
    }
    template <int LeafMode, int Mode, class Stack>
    __device__ static void step(const void *nodes, int64_t n_nodes, const SceneData &ld,
                                const Ray &r, const Prep &, bool fast, Stack &st, State &s,
                                uint32_t &nfetch, uint32_t &ntri, bool &incomplete) {
        if (s.progress()) bin_visit<Node>(nodes, n_nodes, ld, r, fast, st, s, nfetch, incomplete);
        if (s.leaf != kRefEmpty) bin_test_parked<LeafMode, Mode>(ld, r, s, ntri);
    }
    // One round of the two-phase order, as wide_round: lanes visit nodes and
    // park the leaves they meet (one, and one held), then the parked leaves
    // are tested.
    template <int LeafMode, int Mode, class Stack>
    __device__ static void wave(const void *nodes, int64_t n_nodes, const SceneData &ld,
                                const Ray &r, const Prep &, bool fast, bool coherent, Stack &st,
                                State &s, WaveLeafLds *wl, uint32_t &nfetch, uint32_t &ntri,
                                bool &incomplete) {
        for (;;) {
            if (s.progress()) bin_visit<Node>(nodes, n_nodes, ld, r, fast, st, s, nfetch, incomplete);
            const uint64_t prog = __builtin_amdgcn_ballot_w64(s.progress());
            const uint64_t parked = __builtin_amdgcn_ballot_w64(s.leaf != kRefEmpty);
            if (phase_over<kCoherentStall, kStall>(coherent, prog, parked)) break;
        }
        const bool want = s.leaf != kRefEmpty;
        if (coherent) {
            if (want) bin_test_parked<LeafMode, Mode>(ld, r, s, ntri);
            return;
        }
        const uint32_t first = s.leaf >> 5, cnt = ((s.leaf >> 1) & 0xFu) + 1u;
        const bool ended =
            wave_test_leaves<LeafMode, Mode>(ld, r, want, first, cnt, s.best, ntri, wl);
        if (want) bin_tested<Mode>(r, ended, s);
    }
};

template <int Layout>
struct TracerFor;
template <>
struct TracerFor<BVH_LAYOUT_AABB2> {
    using type = BinTracer<BinAABB2>;
};
template <>
struct TracerFor<BVH_LAYOUT_PBRT_Q16> {
    using type = BinTracer<BinPbrtQ16>;
};
template <>
struct TracerFor<BVH_LAYOUT_SG_EQ> {
    using type = BinTracer<BinSgEq>;
};
template <>
struct TracerFor<BVH_LAYOUT_PBRT_SOAOS> {
    using type = BinTracer<BinPbrtSoAoS>;
};
template <>
struct TracerFor<BVH_LAYOUT_PBRT_Q16_SOAOS> {
    using type = BinTracer<BinPbrtQ16SoAoS>;
};
template <>
struct TracerFor<BVH_LAYOUT_SG_EQ_A16> {
    using type = BinTracer<BinSgEqA16>;
};
template <>
struct TracerFor<BVH_LAYOUT_BVH4> {
    using type = WideTracer<DecodeBVH4>;
};
template <>
struct TracerFor<BVH_LAYOUT_BVH8_Q8> {
    using type = WideTracer<DecodeBVH8Q8>;
};
template <>
struct TracerFor<BVH_LAYOUT_BVH8_Q16> {
    using type = WideTracer<DecodeBVH8Q16>;
};

// Whole-ray traversal in one lane.
template <int Layout, int LeafMode, int Mode, class Stack>
__device__ inline Best trace_ray(const void *nodes, int64_t n_nodes, const SceneData &ld,
                                 const Ray &r, Stack &st, uint32_t &nfetch, uint32_t &ntri,
                                 bool &incomplete) {
    using Tr = typename TracerFor<Layout>::type;
    const typename Tr::Prep prep = Tr::prep(r);
    const bool fast = wave_fast(r);
    typename Tr::State s = Tr::start(n_nodes, r);
    while (!Tr::done(s))
        Tr::template step<LeafMode, Mode>(nodes, n_nodes, ld, r, prep, fast, st, s, nfetch, ntri,
                                          incomplete);
    return s.best;
}

constexpr uint32_t kNoRay = 0xFFFFFFFFu;  // ray index of an idle lane

// Work area of the fallback pass: a counter and list of rays that
// overflowed the LDS stack, and one deep stack per fallback lane.
constexpr int kFallbackBlocks = 128;
constexpr int kFallbackLanes = kFallbackBlocks * kTraceBlock;
// The dynamic part of a persistent launch is dealt by kQueues counters, each
// on a line of its own and each handing out one slice of the part: waves
// start at different queues, so their claims do not all serialise on one
// word (device-scope atomics on one address are ordered across the XCDs).
constexpr uint32_t kQueues = 8;
constexpr size_t kQueueStride = 256;  // bytes between two queue counters

struct Fallback {
    uint32_t *count;     // rays appended by the fast pass
    unsigned long long *queue;  // queue q's next unclaimed offset at queue + q * kQueueStride bytes
    uint32_t *list;      // ray indices (capacity: rays of the launch)
    uint64_t *stack;     // [fallback lanes][kStackMax]
};

// Bytes of the header (counter line, queue lines) that must be zero before a launch.
constexpr size_t kFallbackHeaderBytes = kQueueStride * (1 + kQueues);

// Bytes of a work area for n_rays rays and `lanes` fallback lanes (the
// fallback grid's threads).
constexpr size_t fallback_bytes(uint64_t n_rays, size_t lanes = kFallbackLanes) {
    return kFallbackHeaderBytes + ((n_rays * 4 + 7) & ~(uint64_t)7) + lanes * kStackMax * 8;
}

// Carves the work area out of one allocation of fallback_bytes(n_rays, ...).
inline Fallback fallback_view(void *base, uint64_t n_rays) {
    char *p = static_cast<char *>(base);
    Fallback f;
    f.count = reinterpret_cast<uint32_t *>(p);
    f.queue = reinterpret_cast<unsigned long long *>(p + kQueueStride);
    char *q = p + kFallbackHeaderBytes;
    f.list = reinterpret_cast<uint32_t *>(q);
    f.stack = reinterpret_cast<uint64_t *>(q + ((n_rays * 4 + 7) & ~(uint64_t)7));
    return f;
}

// Claims the calling wave's next chunk of `claim` items of the dynamic part
// [static_end, n) (wave-uniform call; `leader` is an active lane): from queue
// q, then from the following queues as they run dry (q is updated).  Returns
// false once all are exhausted, else the chunk [fresh, fresh_end).
__device__ inline bool claim_dynamic(const Fallback &fb, uint64_t static_end, uint64_t n,
                                     uint32_t claim, uint32_t leader, uint32_t &q,
                                     uint64_t &fresh, uint64_t &fresh_end) {
    const uint64_t qlen = (n - static_end + kQueues - 1) / kQueues;
    for (uint32_t tries = 0; tries < kQueues; tries++) {
        const uint64_t qs = static_end + (uint64_t)q * qlen;
        const uint64_t qe = qs + qlen < n ? qs + qlen : n;
        uint32_t lo = 0xFFFFFFFFu, hi = 0x7FFFFFFFu;  // "exhausted" for an empty slice
        if ((threadIdx.x & 63u) == leader && qs < qe) {
            unsigned long long *w = reinterpret_cast<unsigned long long *>(
                reinterpret_cast<char *>(fb.queue) + (size_t)q * kQueueStride);
            const unsigned long long b = atomicAdd(w, (unsigned long long)claim);
            lo = (uint32_t)b;
            hi = (uint32_t)(b >> 32);
        }
        const uint64_t b = ((uint64_t)__builtin_amdgcn_readlane(hi, leader) << 32) |
                           __builtin_amdgcn_readlane(lo, leader);
        if (qs < qe && b < qe - qs) {
            fresh = qs + b;
            fresh_end = fresh + claim < qe ? fresh + claim : qe;
            return true;
        }
        q = (q + 1u) % kQueues;
    }
    return false;
}

// Leaves a ray to the fallback pass; false where the launch has none (no list).
__host__ __device__ inline bool fallback_append(const Fallback &fb, uint32_t ray) {
    if (!fb.count) return false;
    const uint32_t k = __hip_atomic_fetch_add(fb.count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    fb.list[k] = ray;
    return true;
}

// ---------------------------------------------------------------------------
// Host-side launch helpers of the persistent kernels.
// ---------------------------------------------------------------------------
// Per-scene data of a handle for the traversal kernels.  SHARED_SLAB carries
// the scene box (the root's inherited box) in fo (lower) and ft (upper).
inline SceneData scene_data(const bvh_handle_s *h) {
    const bool slab = h->layout == BVH_LAYOUT_SHARED_SLAB;
    const float *lo = slab ? h->scene_lo : h->frame_origin;
    const float *top = slab ? h->scene_hi : h->frame_top;
    return SceneData{h->leaf, h->verts, h->tris, (uint32_t)h->n_tris, h->coord_max(),
                     {lo[0], lo[1], lo[2]},
                     {h->frame_scale[0], h->frame_scale[1], h->frame_scale[2]},
                     {top[0], top[1], top[2]},
                     topo_of(h->nodes, h->n_nodes, h->layout)};
}

// Per-lane stacks of the shared-slab kernels in a global work area: entry e
// of lane l is ref[e * lanes + l] and words box[(e * W + k) * lanes + l],
// k < W, of the box (and, for point queries, distance) it carries.
struct CarriedStack {
    uint32_t *ref;
    float *box;
    uint32_t lanes, cap;
};

// Launch shape of the shared-slab kernels: grid-stride over the queries with
// at most kSlabLanes lanes, each with a stack of cap entries of W words.
constexpr uint32_t kSlabLanes = 131072;
inline int32_t carried_stack(hipStream_t s, uint64_t n, int32_t max_stack, int words,
                             CarriedStack &cs, unsigned &grid) {
    const uint64_t need = (n + kTraceBlock - 1) / kTraceBlock;
    grid = (unsigned)std::min<uint64_t>(need, kSlabLanes / kTraceBlock);
    if (grid == 0) grid = 1;
    cs.lanes = grid * kTraceBlock;
    cs.cap = (uint32_t)(max_stack > 0 ? max_stack : 1) + 1u;
    const size_t ref_bytes = ((size_t)cs.lanes * cs.cap * 4 + 255) & ~(size_t)255;
    void *ws = nullptr;
    BVH_TRY(stream_workspace(s, kAreaTrace, ref_bytes + (size_t)cs.lanes * cs.cap * words * 4, &ws));
    cs.ref = static_cast<uint32_t *>(ws);
    cs.box = reinterpret_cast<float *>(static_cast<char *>(ws) + ref_bytes);
    return BVH_OK;
}
// Spill entries per lane of a persistent launch (beyond the LDS ring).
constexpr uint32_t kSpillCap = 64;

// Workgroups of a kernel resident on one CU at once: the runtime's occupancy
// figure, lowered so that the workgroups' static LDS stays strictly below the
// CU's capacity.  With the LDS of the runtime's figure filling the CU exactly
// (five 32 KiB workgroups in 160 KiB), a persistent grid of that size ran
// about a quarter slower than one a workgroup per CU smaller, as if the last
// workgroup of each CU started only once another had finished (the work
// dealt to it in advance then ends late).
inline int32_t blocks_per_cu(const void *kernel, int dev, int &per_cu) {
    BVH_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kTraceBlock, 0));
    hipFuncAttributes attr;
    BVH_HIP_TRY(hipFuncGetAttributes(&attr, kernel));
    int lds_cu = 0;
    BVH_HIP_TRY(hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev));
    if (attr.sharedSizeBytes > 0 && lds_cu > 0) {
        const int cap = (int)((size_t)(lds_cu - 1) / attr.sharedSizeBytes);
        per_cu = per_cu < cap ? per_cu : cap;
    }
    if (per_cu < 1) per_cu = 1;
    return BVH_OK;
}

// Resident blocks of a kernel on the current device (cached per kernel).
template <typename K>
inline int32_t resident_blocks(K kernel, unsigned &blocks) {
    static std::mutex mu;
    static std::map<std::pair<const void *, int>, unsigned> cache;
    int dev = 0;
    BVH_HIP_TRY(hipGetDevice(&dev));
    const auto key = std::make_pair(reinterpret_cast<const void *>(kernel), dev);
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = cache.find(key);
        if (it != cache.end()) {
            blocks = it->second;
            return BVH_OK;
        }
    }
    int per_cu = 0, n_cu = 0;
    BVH_TRY(blocks_per_cu(reinterpret_cast<const void *>(kernel), dev, per_cu));
    BVH_HIP_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    blocks = (unsigned)per_cu * (unsigned)(n_cu > 0 ? n_cu : 1);
    std::lock_guard<std::mutex> lock(mu);
    cache[key] = blocks;
    return BVH_OK;
}

// Work area of one launch: the fallback header, list and deep stacks, then
// (persistent launches) the per-lane spill area.
struct TraceArea {
    Fallback fb;
    SpillArea sa;
};

// Clears a fallback header: a kernel rather than a memset node, so that the
// call can be captured into a graph.
static __global__ __launch_bounds__(kTraceBlock) void k_zero_words(uint32_t *p, uint32_t n) {
    for (uint32_t k = threadIdx.x; k < n; k += kTraceBlock) p[k] = 0u;
}
inline void clear_header(const Fallback &fb, hipStream_t s) {
    k_zero_words<<<1, kTraceBlock, 0, s>>>(fb.count, (uint32_t)(kFallbackHeaderBytes / 4));
}

// Spill runs of a launch that deals n rays, `claim` at a time, on at most
// `resident` blocks.  Rays spread thin (claim below 64) are dealt in one round, so
// only the first `claim` lanes of a wave ever hold one: the runs are as many as
// the rays, not as the lanes of the grid (30,000 rays: 15 MB, not 168).  Never
// fewer for more rays, so that an area that served a call serves every smaller
// one, also while its stream is captured.
constexpr uint64_t spill_runs(uint64_t n, uint64_t resident) {
    return std::min<uint64_t>(resident * kTraceBlock, (n + kTraceBlock - 1) / kTraceBlock * kTraceBlock + kTraceBlock);
}

inline int32_t trace_area(hipStream_t s, uint64_t n, uint64_t resident, uint32_t claim, TraceArea &ta) {
    const size_t fb_bytes = (fallback_bytes(n) + 255) & ~(size_t)255;
    const size_t sp_bytes = (size_t)spill_runs(n, resident) * kSpillCap * 8;
    void *ws = nullptr;
    BVH_TRY(stream_workspace(s, kAreaTrace, fb_bytes + sp_bytes, &ws));
    ta.fb = fallback_view(ws, n);
    char *sp = static_cast<char *>(ws) + fb_bytes;
    ta.sa.ent = reinterpret_cast<uint64_t *>(sp);
    ta.sa.per_wave = std::min(claim, 64u);
    ta.sa.cap = kSpillCap;
    clear_header(ta.fb, s);
    return BVH_OK;
}

}  // namespace bvhlib
