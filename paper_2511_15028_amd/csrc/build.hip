// GPU construction of the BVH: a linear BVH (Morton order) as the logical
// tree, then packing into one of the node layouts.  The paper fixes the
// topology first and specialises only the physical packing to a layout
// (Sec. 5, two-phase construction); the packing kernels here play the part of
// its generated constructors (count pass, then fill pass, App. F).
#include <algorithm>
#include <array>
#include <cmath>
#include <cstddef>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "internal.h"

namespace bvhlib {
namespace {

constexpr int kBlock = 256;
constexpr int kWave = 64;

struct Box {
    float4 lo;  // w: unused, except in the node boxes (nbox): the node's triangle count
    float4 hi;  // w: unused, except in the node boxes (nbox): its first sorted triangle
};

// The node boxes carry the node's range in their spare words, so a reader of
// a node's box gets its range from the same 32-byte load.
__device__ inline Box with_range(Box b, uint32_t first, uint32_t count) {
    b.lo.w = __uint_as_float(count);
    b.hi.w = __uint_as_float(first);
    return b;
}
__device__ inline uint32_t range_count(const Box &b) { return __float_as_uint(b.lo.w); }
__device__ inline uint32_t range_first(const Box &b) { return __float_as_uint(b.hi.w); }

struct BuildInfo {
    float slo[3], shi[3];   // scene box
    float clo[3], chi[3];   // box of the primitive-box centres
    uint32_t err;           // bit 0: vertex index out of range; bit 1: non-finite extent
    uint32_t n_leaves;      // leaves of the collapsed binary tree
    uint32_t max_depth;     // nodes on the longest root-to-leaf path
    uint32_t max_stack;     // worst-case traversal stack entries
    uint32_t next_count;    // wide packing: size of the next frontier
    uint32_t pad[3];
};

inline unsigned grid_for(uint64_t n, int per_block = kBlock) {
    return (unsigned)((n + per_block - 1) / per_block);
}

// ---------------------------------------------------------------------------
// Wave / block reductions and scans (wave64)
// ---------------------------------------------------------------------------
__device__ inline uint32_t wave_incl_scan(uint32_t v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        uint32_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan of one value per thread over the block (THREADS threads,
// wsum THREADS / kWave words); *total = block sum.
template <int THREADS = kBlock>
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t *total, uint32_t *wsum) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t inc = wave_incl_scan(v);
    if (lane == kWave - 1) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < THREADS / kWave; i++) {
        uint32_t s = wsum[i];
        off += (i < w) ? s : 0u;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

__device__ inline float readlane_t(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline uint32_t readlane_t(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

// Cross-lane steps through DPP (data-parallel primitives of the VALU: one
// instruction each, no LDS traffic).  dpp<CTRL, ROWS>(old, v) gives each lane
// of the written rows the value v of its source lane, or `old` where the
// source is outside the row; GFX9 controls: row_shl:n = 0x100 + n, row_shr:n
// = 0x110 + n, wave_shl:1 = 0x130, row_bcast:15 = 0x142, row_bcast:31 = 0x143.
template <int CTRL, int ROWS, typename T>
__device__ inline T dpp(T old, T v) {
    static_assert(sizeof(T) == 4, "32-bit lanes");
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                             __builtin_bit_cast(int, v), CTRL,
                                                             ROWS, 0xf, false));
}
// Inclusive scan within each 32-lane half (lanes 0-31 and 32-63): within the
// 16-lane rows, then the last lane of rows 0 and 2 into rows 1 and 3.
template <typename T, typename Op>
__device__ inline T half_scan(T v, T id, Op op) {
    v = op(v, dpp<0x111, 0xf>(id, v));
    v = op(v, dpp<0x112, 0xf>(id, v));
    v = op(v, dpp<0x114, 0xf>(id, v));
    v = op(v, dpp<0x118, 0xf>(id, v));
    return op(v, dpp<0x142, 0xa>(id, v));
}
// Inclusive suffix scan within each 32-lane half: within the rows, then the
// first lane of rows 1 and 3 (their row totals by then) into rows 0 and 2.
template <typename T, typename Op>
__device__ inline T half_suffix_scan(T v, T id, Op op, int lane) {
    v = op(v, dpp<0x101, 0xf>(id, v));
    v = op(v, dpp<0x102, 0xf>(id, v));
    v = op(v, dpp<0x104, 0xf>(id, v));
    v = op(v, dpp<0x108, 0xf>(id, v));
    const T r1 = readlane_t(v, 16), r3 = readlane_t(v, 48);
    if (lane < 16) v = op(v, r1);
    else if (lane >= 32 && lane < 48) v = op(v, r3);
    return v;
}
// Whole-wave reduction: the row scans, the two broadcasts, then lane 63.
template <typename T, typename Op>
__device__ inline T wave_reduce(T v, T id, Op op) {
    v = op(v, dpp<0x111, 0xf>(id, v));
    v = op(v, dpp<0x112, 0xf>(id, v));
    v = op(v, dpp<0x114, 0xf>(id, v));
    v = op(v, dpp<0x118, 0xf>(id, v));
    v = op(v, dpp<0x142, 0xa>(id, v));
    v = op(v, dpp<0x143, 0xc>(id, v));
    return readlane_t(v, 63);
}

__device__ inline float wave_min(float v) {
    return wave_reduce<float>(v, INFINITY, [](float a, float b) { return fminf(a, b); });
}
// Orders the wave's LDS accesses before and after it.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Build-wide maxima (stack and depth bounds) without contention: one
// atomicMax per wave into one of kMaxSlots slots chosen by the wave's global
// index, each slot on a cache line of its own, folded by k_fold_max_slots at
// the end.  Device-scope atomics on one word (or one line) from every wave
// of a launch serialise across the XCDs (tens of microseconds per large
// launch); spread over 256 lines they do not.  Every lane of the wave must
// reach the call (lanes with nothing to report pass 0).
constexpr int kMaxSlots = 256;
constexpr int kSlotStride = 32;  // words between slots: one 128-byte line each

__device__ inline void wave_max_to_slots(uint32_t *slots, uint32_t v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, kWave));
    const uint32_t wave = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0 && v)
        atomicMax(&slots[(wave & (kMaxSlots - 1)) * kSlotStride], v);
}

__device__ inline float wave_max(float v) {
    return wave_reduce<float>(v, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
}

// ---------------------------------------------------------------------------
// Exclusive scan of uint32 arrays: per-tile sums, a single-block scan of the
// tile sums, then per-tile scans.  Works in place.
// ---------------------------------------------------------------------------
constexpr int kScanItems = 4;
constexpr int kScanTile = kBlock * kScanItems;

__global__ __launch_bounds__(kBlock) void k_scan_reduce(const uint32_t *in, uint32_t n,
                                                        uint32_t *tile_sums) {
    __shared__ uint32_t wsum[kBlock / kWave];
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++)
        if (base + k < n) s += in[base + k];
    uint32_t tot;
    block_excl_scan(s, &tot, wsum);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kBlock) void k_scan_tiles(uint32_t *tile_sums, uint32_t ntiles,
                                                       uint32_t *total_out) {
    __shared__ uint32_t wsum[kBlock / kWave];
    uint32_t carry = 0;
    for (uint32_t c = 0; c < ntiles; c += kBlock) {
        const uint32_t i = c + threadIdx.x;
        uint32_t v = i < ntiles ? tile_sums[i] : 0u;
        uint32_t tot;
        uint32_t ex = block_excl_scan(v, &tot, wsum);
        if (i < ntiles) tile_sums[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0 && total_out) {
        *total_out = carry;
        __threadfence_system();  // the total may live in host memory the host polls
    }
}

__global__ __launch_bounds__(kBlock) void k_scan_final(const uint32_t *in, uint32_t *out,
                                                       uint32_t n, const uint32_t *tile_sums) {
    __shared__ uint32_t wsum[kBlock / kWave];
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        v[k] = base + k < n ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan(s, &tot, wsum) + tile_sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
}

// Short arrays (a few tiles) in one block: tile after tile with a carry.
constexpr uint32_t kScanSingleTiles = 8;

__global__ __launch_bounds__(kBlock) void k_scan_single(const uint32_t *in, uint32_t *out,
                                                        uint32_t n, uint32_t *total_out) {
    __shared__ uint32_t wsum[kBlock / kWave];
    uint32_t carry = 0;
    for (uint32_t c = 0; c < n; c += kScanTile) {
        const uint32_t base = c + threadIdx.x * kScanItems;
        uint32_t v[kScanItems];
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            v[k] = base + k < n ? in[base + k] : 0u;
            sum += v[k];
        }
        uint32_t tot;
        uint32_t run = carry + block_excl_scan(sum, &tot, wsum);
#pragma unroll
        for (int k = 0; k < kScanItems; k++) {
            if (base + k < n) out[base + k] = run;
            run += v[k];
        }
        carry += tot;
        __syncthreads();  // wsum is reused by the next tile
    }
    if (threadIdx.x == 0 && total_out) {
        *total_out = carry;
        __threadfence_system();  // the total may live in host memory the host polls
    }
}

// Middle-sized arrays: after k_scan_reduce, each block adds up the sums of
// the tiles before it itself (a few thousand at most), so no launch sits
// between the two passes; the last block writes the total.
constexpr uint32_t kScanFusedTiles = 4096;

__global__ __launch_bounds__(kBlock) void k_scan_final_fused(const uint32_t *in, uint32_t *out,
                                                             uint32_t n, const uint32_t *tile_sums,
                                                             uint32_t *total_out) {
    __shared__ uint32_t wsum[kBlock / kWave];
    uint32_t part = 0;
    for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kBlock) part += tile_sums[t];
    uint32_t before;
    block_excl_scan(part, &before, wsum);
    const uint32_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        v[k] = base + k < n ? in[base + k] : 0u;
        sum += v[k];
    }
    uint32_t tot;
    uint32_t run = before + block_excl_scan(sum, &tot, wsum);
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0 && total_out) {
        *total_out = before + tot;
        __threadfence_system();  // the total may live in host memory the host polls
    }
}

// Exclusive scan of n values; total (device) receives the sum if non-null.
// tile_sums must hold ceil(n / kScanTile) entries.
void scan_u32(const uint32_t *in, uint32_t *out, uint32_t n, uint32_t *tile_sums,
              uint32_t *total, hipStream_t s) {
    const uint32_t ntiles = (n + kScanTile - 1) / kScanTile;
    if (ntiles <= kScanSingleTiles) {
        k_scan_single<<<1, kBlock, 0, s>>>(in, out, n, total);
        return;
    }
    if (ntiles <= kScanFusedTiles) {
        k_scan_reduce<<<ntiles, kBlock, 0, s>>>(in, n, tile_sums);
        k_scan_final_fused<<<ntiles, kBlock, 0, s>>>(in, out, n, tile_sums, total);
        return;
    }
    if (ntiles > 0) k_scan_reduce<<<ntiles, kBlock, 0, s>>>(in, n, tile_sums);
    k_scan_tiles<<<1, kBlock, 0, s>>>(tile_sums, ntiles, total);
    if (ntiles > 0) k_scan_final<<<ntiles, kBlock, 0, s>>>(in, out, n, tile_sums);
}

// The clears at the start of a build, in one launch: the build info and the
// slot words set to zero, the leaf marks to zero (layouts that mark leaves)
// and the parent links to -1 (where the topology builder does not write every
// one of them).
__global__ __launch_bounds__(kBlock) void k_build_init(BuildInfo *info, uint32_t *slots,
                                                       uint32_t nslots, uint32_t *mark,
                                                       uint32_t nmark, int32_t *parent,
                                                       uint64_t nparent) {
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < sizeof(BuildInfo) / sizeof(uint32_t)) reinterpret_cast<uint32_t *>(info)[i] = 0u;
    if (i < nslots) slots[i] = 0u;
    if (i < nmark) mark[i] = 0u;
    if (i < nparent) parent[i] = -1;
}

// ---------------------------------------------------------------------------
// a1: triangle boxes, scene box and centre box
// ---------------------------------------------------------------------------
// Each thread boxes kPrimItems triangles (block b covers kPrimItems * kBlock
// consecutive ones), so the single-block final reduction reads few partials.
constexpr int kPrimItems = 4;

__global__ __launch_bounds__(kBlock) void k_prim_bounds(const float *verts, int64_t n_verts,
                                                        const int32_t *tris, uint32_t n,
                                                        Box *pbox, float *partial,
                                                        BuildInfo *info) {
    __shared__ float red[12][kBlock / kWave];
    float v[12] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY,
                   INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int item = 0; item < kPrimItems; item++) {
        const uint32_t i = (blockIdx.x * kPrimItems + item) * kBlock + threadIdx.x;
        float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        float c[3] = {INFINITY, INFINITY, INFINITY}, cm[3] = {-INFINITY, -INFINITY, -INFINITY};
        if (i < n) {
            int32_t idx[3] = {tris[3 * (size_t)i], tris[3 * (size_t)i + 1], tris[3 * (size_t)i + 2]};
            bool ok = true;
            for (int k = 0; k < 3; k++) ok = ok && idx[k] >= 0 && (int64_t)idx[k] < n_verts;
            if (!ok) {
                atomicOr(&info->err, 1u);
                for (int a = 0; a < 3; a++) lo[a] = hi[a] = 0.0f;
            } else {
                for (int k = 0; k < 3; k++) {
                    const float *p = verts + 3 * (size_t)idx[k];
                    for (int a = 0; a < 3; a++) {
                        lo[a] = fminf(lo[a], p[a]);
                        hi[a] = fmaxf(hi[a], p[a]);
                    }
                }
            }
            Box b;
            b.lo = make_float4(lo[0], lo[1], lo[2], 0.0f);
            b.hi = make_float4(hi[0], hi[1], hi[2], 0.0f);
            pbox[i] = b;
            for (int a = 0; a < 3; a++) c[a] = cm[a] = 0.5f * lo[a] + 0.5f * hi[a];
        }
        for (int a = 0; a < 3; a++) {
            v[a] = fminf(v[a], lo[a]);
            v[3 + a] = fmaxf(v[3 + a], hi[a]);
            v[6 + a] = fminf(v[6 + a], c[a]);
            v[9 + a] = fmaxf(v[9 + a], cm[a]);
        }
    }
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    for (int k = 0; k < 12; k++) {
        bool is_min = (k < 3) || (k >= 6 && k < 9);
        float r = is_min ? wave_min(v[k]) : wave_max(v[k]);
        if (lane == 0) red[k][w] = r;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
        const int k = threadIdx.x;
        bool is_min = (k < 3) || (k >= 6 && k < 9);
        float r = red[k][0];
        for (int j = 1; j < kBlock / kWave; j++) r = is_min ? fminf(r, red[k][j]) : fmaxf(r, red[k][j]);
        partial[12 * (size_t)blockIdx.x + k] = r;
    }
}

// The workgroups' partial bounds to the scene's, in info and in out (12 words
// of LDS).  Every thread of the block calls it.
template <int THREADS>
__device__ inline void fold_bounds(const float *partial, uint32_t nparts, BuildInfo *info,
                                   float (*red)[THREADS / kWave], float *out) {
    float v[12];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        bool is_min = (k < 3) || (k >= 6 && k < 9);
        v[k] = is_min ? INFINITY : -INFINITY;
    }
    for (uint32_t p = threadIdx.x; p < nparts; p += THREADS)
#pragma unroll
        for (int k = 0; k < 12; k++) {
            bool is_min = (k < 3) || (k >= 6 && k < 9);
            float x = partial[12 * (size_t)p + k];
            v[k] = is_min ? fminf(v[k], x) : fmaxf(v[k], x);
        }
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        bool is_min = (k < 3) || (k >= 6 && k < 9);
        float r = is_min ? wave_min(v[k]) : wave_max(v[k]);
        if (lane == 0) red[k][w] = r;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
        const int k = threadIdx.x;
        bool is_min = (k < 3) || (k >= 6 && k < 9);
        float r = red[k][0];
        for (int j = 1; j < THREADS / kWave; j++) r = is_min ? fminf(r, red[k][j]) : fmaxf(r, red[k][j]);
        out[k] = r;
        if (k < 3) info->slo[k] = r;
        else if (k < 6) info->shi[k - 3] = r;
        else if (k < 9) info->clo[k - 6] = r;
        else info->chi[k - 9] = r;
    }
    __syncthreads();
}

__global__ __launch_bounds__(kBlock) void k_bounds_final(const float *partial, uint32_t nparts,
                                                         BuildInfo *info) {
    __shared__ float red[12][kBlock / kWave];
    __shared__ float out[12];
    fold_bounds<kBlock>(partial, nparts, info, red, out);
}

// ---------------------------------------------------------------------------
// a2: Morton codes of the box centres, `bits` bits per axis (at most 21).
// The builder uses ceil(log2(n)/3) + 4 bits (one less where that saves a
// sort pass): 2^9 to 2^12 grid cells per triangle, so equal codes are rare,
// and the radix sort only sorts 3*bits bits (four 8-bit passes for two
// million triangles instead of eight).
// ---------------------------------------------------------------------------
__device__ inline uint32_t quantize_axis_bits(float x, float lo, float inv_ext, int bits) {
    const float cells = (float)(1u << bits);
    float u = (x - lo) * inv_ext * cells;
    u = fminf(fmaxf(u, 0.0f), cells - 1.0f);
    return (uint32_t)u;
}

// The key of one box; clo and chi bound the box centres.
__device__ inline uint64_t morton_key(const Box &b, const float *clo, const float *chi, int bits) {
    float c[3] = {0.5f * b.lo.x + 0.5f * b.hi.x, 0.5f * b.lo.y + 0.5f * b.hi.y,
                  0.5f * b.lo.z + 0.5f * b.hi.z};
    uint32_t q[3];
    for (int a = 0; a < 3; a++) {
        float ext = chi[a] - clo[a];
        float inv = ext > 0.0f ? 1.0f / ext : 0.0f;
        q[a] = quantize_axis_bits(c[a], clo[a], inv, bits);
    }
    // bit k of x, y, z goes to key bit 3k+2, 3k+1, 3k
    uint64_t key = 0;
    for (int bit = 0; bit < bits; bit++) {
        key |= (uint64_t)((q[0] >> bit) & 1u) << (3 * bit + 2);
        key |= (uint64_t)((q[1] >> bit) & 1u) << (3 * bit + 1);
        key |= (uint64_t)((q[2] >> bit) & 1u) << (3 * bit);
    }
    return key;
}

template <typename KeyT>
__global__ __launch_bounds__(kBlock) void k_morton(const Box *pbox, uint32_t n,
                                                   const BuildInfo *info, int bits,
                                                   KeyT *keys, uint32_t *vals) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    // 3 * bits <= the key width (checked by the caller)
    keys[i] = (KeyT)morton_key(pbox[i], info->clo, info->chi, bits);
    vals[i] = i;
}

inline int morton_bits(int n) {
    int lg = 0;
    while ((1ll << lg) < (long long)std::max(n, 2)) lg++;
    const int b = std::min(21, std::max(4, (lg + 2) / 3 + 4));
    // one bit per axis less when the last 8-bit sort pass would only sort
    // 1-3 bits (33 bits for two million triangles: 4 passes instead of 5;
    // still 2^9 grid cells per triangle, and the traversal times measured the same)
    const int r = (3 * b) % 8;
    return (r >= 1 && r <= 3 && b > 4) ? b - 1 : b;
}

// ---------------------------------------------------------------------------
// a3: stable LSD radix sort of (u64 key, u32 value), 8 bits per pass.
// Per pass three launches: per-tile digit counts (digit-major matrix), one
// block per digit turning its row into exclusive prefixes over the tiles
// plus the digit's total, and the scatter.  The scatter ranks its tile's
// keys stably in LDS (each wave a contiguous quarter of the tile, equal
// digits found with ballots, no block barrier per round), then writes the
// tile out in local digit order, so consecutive lanes store consecutive
// addresses of a digit's run.
// ---------------------------------------------------------------------------
constexpr int kSortItems = 8;
constexpr int kSortTile = kBlock * kSortItems;
constexpr int kSortWaves = kBlock / kWave;
constexpr int kRadix = 256;
static_assert(kRadix == kBlock, "one digit per thread in the per-digit steps");

template <typename KeyT>
__global__ __launch_bounds__(kBlock) void k_radix_hist(const KeyT *keys, uint32_t n, int shift,
                                                       uint32_t *hist, uint32_t ntiles) {
    __shared__ uint32_t h[kRadix];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t base = blockIdx.x * kSortTile;
    for (int k = 0; k < kSortItems; k++) {
        uint32_t i = base + k * kBlock + threadIdx.x;
        if (i < n) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & (kRadix - 1)], 1u);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// Block d: row d of the count matrix -> exclusive prefix over tiles, in
// place; total[d] = the row's sum.
__global__ __launch_bounds__(kBlock) void k_radix_offsets(uint32_t *hist, uint32_t ntiles,
                                                          uint32_t *total) {
    __shared__ uint32_t wsum[kBlock / kWave];
    uint32_t *row = hist + (size_t)blockIdx.x * ntiles;
    uint32_t carry = 0;
    for (uint32_t c = 0; c < ntiles; c += kBlock) {
        const uint32_t t = c + threadIdx.x;
        const uint32_t v = t < ntiles ? row[t] : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan(v, &tot, wsum);
        if (t < ntiles) row[t] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// Moves a wave's keys (row r of the lane: position first + r * 64) to their
// places in the sorted order of one digit, stably: run[d] is the place of the
// wave's next key of digit d.
template <int ROWS, typename KeyT, typename ValT>
__device__ inline void rank_rows(const KeyT (&key)[ROWS], const uint32_t (&val)[ROWS], int rows,
                                 uint32_t first, uint32_t n, int shift, uint32_t *run, KeyT *skey,
                                 ValT *sval) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
#pragma unroll
    for (int r = 0; r < ROWS; r++) {
        if (r >= rows) break;  // the same in the wave
        const bool valid = first + r * kWave < n;
        const uint32_t d = (uint32_t)(key[r] >> shift) & (kRadix - 1);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t start = valid ? run[d] : 0u;
        __builtin_amdgcn_wave_barrier();
        if (valid) {
            const uint32_t pos = start + (uint32_t)__popcll(peers & lt_mask);
            skey[pos] = key[r];
            sval[pos] = (ValT)val[r];
            if ((peers & lt_mask) == 0) run[d] = start + (uint32_t)__popcll(peers);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <typename KeyT>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(const KeyT *keys_in,
                                                          const uint32_t *vals_in,
                                                          KeyT *keys_out, uint32_t *vals_out,
                                                          uint32_t n, int shift,
                                                          const uint32_t *prefix,
                                                          const uint32_t *total,
                                                          uint32_t ntiles) {
    __shared__ KeyT skey[kSortTile];
    __shared__ uint32_t sval[kSortTile];
    __shared__ uint32_t wcount[kSortWaves][kRadix];  // digit counts per wave, then run positions
    __shared__ uint32_t gdst[kRadix];                 // output index of local position 0 of digit d
    __shared__ uint32_t wsum[kBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t tile = blockIdx.x;
    const uint32_t base = tile * kSortTile;
    const uint32_t wbase = base + (uint32_t)w * (kSortItems * kWave);
#pragma unroll
    for (int k = 0; k < kSortWaves; k++) wcount[k][threadIdx.x] = 0;
    __syncthreads();
    // this wave's quarter of the tile, item r of a lane at wbase + r*64 + lane
    KeyT key[kSortItems];
    uint32_t val[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        const uint32_t i = wbase + r * kWave + lane;
        key[r] = i < n ? keys_in[i] : (KeyT)0;
        val[r] = i < n ? vals_in[i] : 0u;
        if (i < n) atomicAdd(&wcount[w][(uint32_t)(key[r] >> shift) & (kRadix - 1)], 1u);
    }
    __syncthreads();
    {   // thread d: local start of digit d per wave, and its output offset
        const uint32_t d = threadIdx.x;
        uint32_t c[kSortWaves], sum = 0;
#pragma unroll
        for (int k = 0; k < kSortWaves; k++) {
            c[k] = wcount[k][d];
            sum += c[k];
        }
        uint32_t tot_local;
        const uint32_t lstart = block_excl_scan(sum, &tot_local, wsum);
        uint32_t tot_all;
        const uint32_t gstart = block_excl_scan(total[d], &tot_all, wsum);
        gdst[d] = gstart + prefix[(size_t)d * ntiles + tile] - lstart;
        uint32_t run = lstart;
#pragma unroll
        for (int k = 0; k < kSortWaves; k++) {
            wcount[k][d] = run;
            run += c[k];
        }
    }
    __syncthreads();
    rank_rows<kSortItems>(key, val, kSortItems, wbase + lane, n, shift, wcount[w], skey, sval);
    __syncthreads();
    const uint32_t m = min((uint32_t)kSortTile, n - base);
    for (uint32_t p = threadIdx.x; p < m; p += kBlock) {
        const KeyT k = skey[p];
        const uint32_t o = gdst[(uint32_t)(k >> shift) & (kRadix - 1)] + p;
        if (o < n) {  // always true for a consistent histogram; guards the write
            keys_out[o] = k;
            vals_out[o] = sval[p];
        }
    }
}

// ---------------------------------------------------------------------------
// a4: hierarchy of the sorted codes (Karras 2012).  Internal node i covers a
// key range [first, last] and splits it at the highest differing bit; equal
// keys are separated by their positions.  Node ids: internal i -> i, sorted
// leaf j -> (n - 1) + j; the root is id 0.
// ---------------------------------------------------------------------------
// Sorted keys as seen by one block: keys [w0, w0 + kKarrasWindow) staged in
// LDS (the block's own nodes and a halo on either side, where nearly all of
// the searches land), the rest read from global memory.
constexpr int kKarrasHalo = 512;
constexpr int kKarrasWindow = kBlock + 2 * kKarrasHalo;

template <typename KeyT>
struct KeyWindow {
    const KeyT *g;
    const KeyT *lds;
    int w0, len;
    __device__ KeyT at(int j) const {
        const unsigned k = (unsigned)(j - w0);
        return k < (unsigned)len ? lds[k] : g[j];
    }
};

// Length of the common prefix of sorted keys i and j (positions i and j
// appended as tie-breaks), -1 when j is out of range.
__device__ inline int prefix_len(uint64_t a, uint64_t b, int i, int j) {
    if (a != b) return __clzll((long long)(a ^ b));
    return 64 + __clz((int)((uint32_t)i ^ (uint32_t)j));
}
__device__ inline int prefix_len(uint32_t a, uint32_t b, int i, int j) {
    if (a != b) return __clz((int)(a ^ b));
    return 32 + __clz((int)((uint32_t)i ^ (uint32_t)j));
}
template <typename KeyT>
__device__ inline int common_prefix(const KeyWindow<KeyT> &kw, KeyT ki, int n, int i, int j) {
    if (j < 0 || j >= n) return -1;
    return prefix_len(ki, kw.at(j), i, j);
}

// Node i of the hierarchy; returns how many leaves of the collapsed tree it
// accounts for (see k_karras).
template <typename KeyT>
__device__ inline uint32_t karras_node(const KeyWindow<KeyT> &kw, int n, int i, int32_t *ileft,
                                       int32_t *iright, uint32_t *ifirst, uint32_t *icount,
                                       uint8_t *iaxis, int32_t *parent, int L) {
    const KeyT ki = kw.at(i);
    const int d = (common_prefix(kw, ki, n, i, i + 1) - common_prefix(kw, ki, n, i, i - 1)) >= 0 ? 1 : -1;
    const int dmin = common_prefix(kw, ki, n, i, i - d);
    int lmax = 2;
    while (common_prefix(kw, ki, n, i, i + lmax * d) > dmin) lmax *= 2;
    int l = 0;
    for (int t = lmax / 2; t >= 1; t /= 2)
        if (common_prefix(kw, ki, n, i, i + (l + t) * d) > dmin) l += t;
    const int j = i + l * d;
    const int dnode = common_prefix(kw, ki, n, i, j);
    int s = 0, t = l;
    do {
        t = (t + 1) >> 1;
        if (common_prefix(kw, ki, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int gamma = i + s * d + (d < 0 ? -1 : 0);
    const int first = min(i, j), last = max(i, j);
    const int lc = (first == gamma) ? (n - 1) + gamma : gamma;
    const int rc = (last == gamma + 1) ? (n - 1) + gamma + 1 : gamma + 1;
    ileft[i] = lc;
    iright[i] = rc;
    parent[lc] = i;
    parent[rc] = i;
    ifirst[i] = (uint32_t)first;
    icount[i] = (uint32_t)(last - first + 1);
    // split axis: key bit (width - 1) - dnode (bit 3b+2 is x, 3b+1 is y, 3b is z)
    constexpr int kKeyBits = 8 * (int)sizeof(KeyT);
    uint8_t axis = 0;
    if (dnode < kKeyBits) {
        const int p = (kKeyBits - 1) - dnode;
        axis = (p % 3 == 2) ? 0 : (p % 3 == 1 ? 1 : 2);
    }
    iaxis[i] = axis;
    if (i == 0) parent[0] = -1;
    const int cnt = last - first + 1, cl = gamma - first + 1, cr = last - gamma;
    if (cnt > L) return (uint32_t)(cl <= L) + (uint32_t)(cr <= L);
    return (i == 0) ? 1u : 0u;  // the root of at most L primitives is the only leaf
}

// With leaf_slots (the wide layouts): also counts the collapsed tree's leaves
// (leaf size L), which are the children of at most L primitives of the nodes
// of more than L, or the root alone when it holds at most L; per-wave counts
// are added into the kMaxSlots slots a line apart, as in k_count_leaves.
template <typename KeyT>
__global__ __launch_bounds__(kBlock) void k_karras(const KeyT *keys, int n, int32_t *ileft,
                                                   int32_t *iright, uint32_t *ifirst,
                                                   uint32_t *icount, uint8_t *iaxis,
                                                   int32_t *parent, int L, uint32_t *leaf_slots) {
    __shared__ KeyT sk[kKarrasWindow];
    const int w0 = (int)(blockIdx.x * kBlock) - kKarrasHalo;
    for (int k = threadIdx.x; k < kKarrasWindow; k += kBlock) {
        const int j = w0 + k;
        if (j >= 0 && j < n) sk[k] = keys[j];
    }
    __syncthreads();
    const KeyWindow<KeyT> kw{keys, sk, w0, kKarrasWindow};
    const int i = blockIdx.x * kBlock + threadIdx.x;
    uint32_t leaves = 0;
    if (i < n - 1) leaves = karras_node(kw, n, i, ileft, iright, ifirst, icount, iaxis, parent, L);
    if (leaf_slots) {  // every lane of the wave arrives here
        const uint32_t c = (uint32_t)__popcll(__ballot(leaves >= 1)) + (uint32_t)__popcll(__ballot(leaves >= 2));
        const uint32_t wave = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
        if ((threadIdx.x & (kWave - 1)) == 0 && c)
            atomicAdd(&leaf_slots[(wave & (kMaxSlots - 1)) * kSlotStride], c);
    }
}


// Small meshes: the scene bounds, the keys, the whole sort and the hierarchy in
// one workgroup with the keys in LDS.  Apart they are 12 launches of 2 to 8 us
// (three of them per sort pass), each a chain of loads that a single workgroup
// of work does not hide.  Builds of 300 / 1,024 / 2,048 / 4,096 triangles 177 /
// 168 / 160 / 160 us apart, 137 / 127 / 123 / 147 together; of 8,192 166 and 179,
// so the line lies where the gain ends.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr uint32_t kSmallMax = 4096;
constexpr int kSmallRows = kSmallMax / kSmallThreads;
static_assert(kSmallMax == kSmallThreads * kSmallRows && kSmallMax <= 65536, "positions in 16 bits");

__global__ __launch_bounds__(kSmallThreads) void k_small_hierarchy(
    const Box *pbox, uint32_t n, const float *partial, uint32_t nparts, BuildInfo *info, int bits,
    uint32_t *perm, int32_t *ileft, int32_t *iright, uint32_t *ifirst, uint32_t *icount,
    uint8_t *iaxis, int32_t *parent, int L, uint32_t *leaf_word) {
    __shared__ uint32_t skey[kSmallMax];
    __shared__ uint16_t sval[kSmallMax];
    __shared__ uint32_t wcount[kSmallWaves][kRadix];
    __shared__ uint32_t wsum[kSmallWaves];
    __shared__ float red[12][kSmallWaves];
    __shared__ float bounds[12];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    // each wave holds consecutive rows of 64 primitives
    const int rows = (int)((n + kSmallThreads - 1) / kSmallThreads);
    const uint32_t first = (uint32_t)(w * rows) * kWave + lane;
    uint32_t key[kSmallRows], val[kSmallRows];
    fold_bounds<kSmallThreads>(partial, nparts, info, red, bounds);
#pragma unroll
    for (int r = 0; r < kSmallRows; r++) {
        key[r] = 0;
        val[r] = first + r * kWave;
        if (r < rows && val[r] < n) key[r] = (uint32_t)morton_key(pbox[val[r]], bounds + 6, bounds + 9, bits);
    }
    for (int shift = 0; shift < 3 * bits; shift += 8) {
        for (int k = threadIdx.x; k < kSmallWaves * kRadix; k += kSmallThreads) wcount[0][k] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallRows; r++)
            if (r < rows && first + r * kWave < n) atomicAdd(&wcount[w][(key[r] >> shift) & (kRadix - 1)], 1u);
        __syncthreads();
        // thread d: the place of digit d's first key per wave
        uint32_t sum = 0, tot;
        if (threadIdx.x < kRadix)
            for (int k = 0; k < kSmallWaves; k++) sum += wcount[k][threadIdx.x];
        uint32_t run = block_excl_scan<kSmallThreads>(sum, &tot, wsum);
        if (threadIdx.x < kRadix)
            for (int k = 0; k < kSmallWaves; k++) {
                const uint32_t c = wcount[k][threadIdx.x];
                wcount[k][threadIdx.x] = run;
                run += c;
            }
        __syncthreads();
        rank_rows<kSmallRows>(key, val, rows, first, n, shift, wcount[w], skey, sval);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallRows; r++) {
            const uint32_t i = first + r * kWave;
            if (r >= rows || i >= n) break;
            key[r] = skey[i];
            val[r] = sval[i];
        }
    }
#pragma unroll
    for (int r = 0; r < kSmallRows; r++)
        if (r < rows && first + r * kWave < n) perm[first + r * kWave] = val[r];
    const KeyWindow<uint32_t> kw{nullptr, skey, 0, (int)n};
    uint32_t leaves = 0;
    for (int i = threadIdx.x; i < (int)n - 1; i += kSmallThreads)
        leaves += karras_node(kw, (int)n, i, ileft, iright, ifirst, icount, iaxis, parent, L);
    if (leaf_word) {  // the collapsed tree's leaves, as k_karras counts them
        uint32_t total;
        block_excl_scan<kSmallThreads>(leaves, &total, wsum);
        if (threadIdx.x == 0) {
            *leaf_word = total;
            __threadfence_system();  // the host polls the word
        }
    }
}

// ---------------------------------------------------------------------------
// a5: node boxes.  Every node of the hierarchy covers a contiguous range of
// the sorted primitives, so its box is the union of the primitive boxes in
// that range: a range query, answered without any inter-thread
// synchronisation.  Sorted primitive boxes are grouped in blocks of kRangeBlock;
// a sparse table holds the union of 2^k consecutive blocks, so a range is
// its partial blocks (read directly) plus at most two overlapping table
// entries (min/max are idempotent).
// ---------------------------------------------------------------------------
constexpr int kRangeBlock = 64;

__device__ inline Box box_union(const Box &a, const Box &b) {
    Box u;
    u.lo = make_float4(fminf(a.lo.x, b.lo.x), fminf(a.lo.y, b.lo.y), fminf(a.lo.z, b.lo.z), 0.0f);
    u.hi = make_float4(fmaxf(a.hi.x, b.hi.x), fmaxf(a.hi.y, b.hi.y), fmaxf(a.hi.z, b.hi.z), 0.0f);
    return u;
}

__device__ inline Box box_empty() {
    Box e;
    e.lo = make_float4(INFINITY, INFINITY, INFINITY, 0.0f);
    e.hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.0f);
    return e;
}

// Leaf boxes in sorted order (node ids n-1 .. 2n-2) and, one wave per block
// of kRangeBlock: the block union (sparse-table level 0) and the in-block
// prefix and suffix unions (inclusive wave scans).
__device__ inline void wave_scan_box(float *v, bool reverse) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const float t = reverse ? __shfl_down(v[k], o, kWave) : __shfl_up(v[k], o, kWave);
            const bool take = reverse ? (lane + o < kWave) : (lane >= o);
            if (take) v[k] = k < 3 ? fminf(v[k], t) : fmaxf(v[k], t);
        }
    }
}

__device__ inline Box box_of(const float *v) {
    Box u;
    u.lo = make_float4(v[0], v[1], v[2], 0.0f);
    u.hi = make_float4(v[3], v[4], v[5], 0.0f);
    return u;
}

__global__ __launch_bounds__(kBlock) void k_leaf_boxes(const Box *pbox, const uint32_t *perm, int n,
                                                       Box *nbox, Box *table, Box *pre, Box *suf) {
    const int j = blockIdx.x * kBlock + threadIdx.x;
    Box b = box_empty();
    if (j < n) {
        b = pbox[perm[j]];
        nbox[(n - 1) + j] = with_range(b, (uint32_t)j, 1u);
    }
    const float v0[6] = {b.lo.x, b.lo.y, b.lo.z, b.hi.x, b.hi.y, b.hi.z};
    float p[6], q[6];
    for (int k = 0; k < 6; k++) p[k] = q[k] = v0[k];
    wave_scan_box(p, false);
    wave_scan_box(q, true);
    if (j < n) {
        pre[j] = box_of(p);
        suf[j] = box_of(q);
    }
    const int blk = j / kRangeBlock;
    if ((threadIdx.x & (kWave - 1)) == kWave - 1 && blk * kRangeBlock < n) table[blk] = box_of(p);
}

// Sparse-table levels k0 .. k0+m-1 (m <= 3) from level k0-1 in one launch:
// T_{k0-1+d}[i] = union over j < 2^d of T_{k0-1}[i + j 2^(k0-1)], written
// where the entry's 2^(k0-1+d) blocks lie inside the table.
__global__ __launch_bounds__(kBlock) void k_table_levels(Box *table, int nblocks, int k0, int m) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int half = 1 << (k0 - 1);
    const Box *base = table + (size_t)(k0 - 1) * nblocks;
    Box u = box_empty();
    for (int d = 1; d <= m; d++) {
        if (i + (half << d) > nblocks) return;
        // fold in the entries j in [2^(d-1), 2^d)
        for (int j = (d == 1 ? 0 : 1 << (d - 1)); j < (1 << d); j++) u = box_union(u, base[i + j * half]);
        table[(size_t)(k0 - 1 + d) * nblocks + i] = u;
    }
}

// Internal node i's range has i as one end (Karras order) or contains it
// (the SAH ids), so a range inside one 64-block lies within 64 leaves of i:
// the workgroup stages the leaf boxes around its nodes in LDS (coalesced,
// about 1.5 boxes per node) and unions in-block ranges from there, whole groups
// of kBoxGroup boxes at a time (a wave's longest range is 8 + 6 + 8 steps
// instead of 64: 1,024 triangles 10.3 -> 6.2 us, 2.1 M 57 -> 50 us); a range
// outside the window (the SAH root's remapped id) reads global memory.
constexpr int kBoxWindow = kBlock + 2 * kRangeBlock;
constexpr int kBoxGroup = 8;
static_assert(kBoxWindow % kBoxGroup == 0 && kRangeBlock % kBoxGroup == 0, "whole groups in a window");

__global__ __launch_bounds__(kBlock) void k_internal_boxes(const uint32_t *ifirst,
                                                           const uint32_t *icount, int n,
                                                           const Box *table, int nblocks,
                                                           const Box *pre, const Box *suf,
                                                           Box *nbox, float *area) {
    __shared__ float wb[6][kBoxWindow];
    __shared__ float gb[6][kBoxWindow / kBoxGroup];
    const int i0 = blockIdx.x * kBlock;
    const int wlo = max(0, i0 - kRangeBlock), whi = min(n, i0 + kBlock + kRangeBlock);
    const Box *leaf = nbox + (n - 1);
    for (int j = wlo + (int)threadIdx.x; j < whi; j += kBlock) {
        const Box x = leaf[j];
        wb[0][j - wlo] = x.lo.x;
        wb[1][j - wlo] = x.lo.y;
        wb[2][j - wlo] = x.lo.z;
        wb[3][j - wlo] = x.hi.x;
        wb[4][j - wlo] = x.hi.y;
        wb[5][j - wlo] = x.hi.z;
    }
    __syncthreads();
    // (a group that the window's end cuts short is never used)
    for (int k = threadIdx.x; k < 6 * (kBoxWindow / kBoxGroup); k += kBlock) {
        const int c = k % 6, g = k / 6;
        float v = wb[c][g * kBoxGroup];
#pragma unroll
        for (int j = 1; j < kBoxGroup; j++) {
            const float x = wb[c][g * kBoxGroup + j];
            v = c < 3 ? fminf(v, x) : fmaxf(v, x);
        }
        gb[c][g] = v;
    }
    __syncthreads();
    const int i = i0 + (int)threadIdx.x;
    if (i >= n - 1) return;
    const int a = (int)ifirst[i], b = a + (int)icount[i] - 1;
    if (a < 0 || b >= n || b < a) {  // malformed range: empty box, the range as given
        nbox[i] = with_range(box_empty(), ifirst[i], icount[i]);
        return;
    }
    const int ba = a / kRangeBlock, bb = b / kRangeBlock;
    Box u = box_empty();
    if (ba == bb && a >= wlo && b < whi) {
        float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
        // [ja, jb): single boxes up to the first whole group and from the last one on
        const int ja = a - wlo, jb = b - wlo + 1;
        const int g0 = (ja + kBoxGroup - 1) / kBoxGroup, g1 = jb / kBoxGroup;
        const int head = g0 < g1 ? g0 * kBoxGroup : jb, tail = g0 < g1 ? g1 * kBoxGroup : jb;
        for (int j = ja; j < head; j++) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                v[c] = fminf(v[c], wb[c][j]);
                v[3 + c] = fmaxf(v[3 + c], wb[3 + c][j]);
            }
        }
        for (int g = g0; g < g1; g++) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                v[c] = fminf(v[c], gb[c][g]);
                v[3 + c] = fmaxf(v[3 + c], gb[3 + c][g]);
            }
        }
        for (int j = tail; j < jb; j++) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                v[c] = fminf(v[c], wb[c][j]);
                v[3 + c] = fmaxf(v[3 + c], wb[3 + c][j]);
            }
        }
        u.lo = make_float4(v[0], v[1], v[2], 0.0f);
        u.hi = make_float4(v[3], v[4], v[5], 0.0f);
    } else if (ba == bb) {
        int j = a;
        for (; j + 3 <= b; j += 4) {
            const Box x0 = leaf[j], x1 = leaf[j + 1], x2 = leaf[j + 2], x3 = leaf[j + 3];
            u = box_union(u, box_union(box_union(x0, x1), box_union(x2, x3)));
        }
        for (; j <= b; j++) u = box_union(u, leaf[j]);
    } else {
        // suffix of a's block, prefix of b's block, whole blocks in between
        u = box_union(suf[a], pre[b]);
        const int lo = ba + 1, hi = bb - 1;
        if (lo <= hi) {
            const int len = hi - lo + 1;
            const int k = 31 - __clz(len);
            const Box *lvl = table + (size_t)k * nblocks;
            u = box_union(u, box_union(lvl[lo], lvl[hi - (1 << k) + 1]));
        }
    }
    nbox[i] = with_range(u, (uint32_t)a, (uint32_t)(b - a + 1));
    const float dx = u.hi.x - u.lo.x, dy = u.hi.y - u.lo.y, dz = u.hi.z - u.lo.z;
    area[i] = dx * dy + dy * dz + dz * dx;
}

// ---------------------------------------------------------------------------
// a6: collapse.  A node is kept ("alive") if it is the root or its parent
// holds more than L triangles; an alive node with at most L triangles is a
// leaf covering its sorted range.  mark[first] = 1 for every leaf.
// ---------------------------------------------------------------------------
struct TreeView {
    int n;                 // triangles
    int leaf_size;
    const int32_t *ileft, *iright, *parent;
    const uint32_t *ifirst, *icount;
    const uint8_t *iaxis;
    const Box *nbox;
    const float *area;     // surface-area measure of internal nodes
    uint32_t *stack_slots;  // kMaxSlots slots each, kSlotStride words apart (zeroed at build start): see wave_max_to_slots
    uint32_t *depth_slots;
    __device__ bool is_prim(int x) const { return x >= n - 1; }
    __device__ uint32_t count(int x) const { return is_prim(x) ? 1u : icount[x]; }
    __device__ uint32_t first(int x) const { return is_prim(x) ? (uint32_t)(x - (n - 1)) : ifirst[x]; }
    __device__ bool alive(int x) const {
        if (x == 0) return true;
        const int p = parent[x];
        return p >= 0 && p < n - 1 && icount[p] > (uint32_t)leaf_size;
    }
    __device__ bool is_leaf(int x) const { return count(x) <= (uint32_t)leaf_size; }
};

__global__ __launch_bounds__(kBlock) void k_mark_leaves(TreeView tv, uint32_t *mark) {
    const int x = blockIdx.x * kBlock + threadIdx.x;
    if (x >= 2 * tv.n - 1) return;
    if (tv.alive(x) && tv.is_leaf(x)) mark[tv.first(x)] = 1u;
}

// The wide layouts need only the number of leaves: per-wave counts added
// into kMaxSlots slots a line apart, then folded into a host-mapped word.
__global__ __launch_bounds__(kBlock) void k_count_leaves(TreeView tv, uint32_t *slots) {
    const int x = blockIdx.x * kBlock + threadIdx.x;
    const bool leaf = x < 2 * tv.n - 1 && tv.alive(x) && tv.is_leaf(x);
    const uint64_t b = __ballot(leaf);
    const uint32_t wave = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0 && b)
        atomicAdd(&slots[(wave & (kMaxSlots - 1)) * kSlotStride], (uint32_t)__popcll(b));
}

__global__ __launch_bounds__(kBlock) void k_fold_leaf_count(const uint32_t *slots, uint32_t *host_word) {
    __shared__ uint32_t wsum[kBlock / kWave];
    uint32_t v = 0;
    for (int i = threadIdx.x; i < kMaxSlots; i += kBlock) v += slots[i * kSlotStride];
    uint32_t total;
    block_excl_scan(v, &total, wsum);
    if (threadIdx.x == 0) {
        *host_word = total;
        __threadfence_system();  // the host polls the word
    }
}

// ---------------------------------------------------------------------------
// a7 (AABB2): preorder packing.  With leaf_before(x) = number of leaves that
// precede x's range (exclusive scan of mark) and lturns(x) = number of
// left-child steps on the root-to-x path, the preorder index of x in the
// collapsed tree is lturns(x) + 2 * leaf_before(x), and the right child of
// interior x sits 2 * (leaf_before(right) - leaf_before(x)) after x.
// ---------------------------------------------------------------------------
// Writes node x's record; reports its depth and, for a leaf, its stack need.
__device__ inline void emit_aabb2_item(const TreeView &tv, int x, const uint32_t *lbefore,
                                       bvh_node_aabb2 *nodes, uint32_t n_nodes, BuildInfo *info,
                                       uint32_t *depth_out, uint32_t *stack_out) {
    uint32_t lturns = 0, depth = 1;
    for (int y = x; y != 0; depth++) {
        const int p = tv.parent[y];
        if (p < 0 || p >= tv.n - 1 || depth >= 1024) {
            atomicOr(&info->err, 4u);
            return;
        }
        lturns += (tv.ileft[p] == y) ? 1u : 0u;
        y = p;
    }
    const uint32_t f = tv.first(x);
    const uint32_t idx = lturns + 2u * lbefore[f];
    if (idx >= n_nodes) {
        atomicOr(&info->err, 4u);
        return;
    }
    bvh_node_aabb2 nd;
    const Box b = tv.nbox[x];
    nd.lo[0] = b.lo.x; nd.lo[1] = b.lo.y; nd.lo[2] = b.lo.z;
    nd.hi[0] = b.hi.x; nd.hi[1] = b.hi.y; nd.hi[2] = b.hi.z;
    if (tv.is_leaf(x)) {
        nd.offset = f;
        nd.meta = tv.count(x);
    } else {
        const int r = tv.iright[x];
        nd.offset = 2u * (lbefore[tv.first(r)] - lbefore[f]);
        nd.meta = (uint32_t)tv.iaxis[x] << 16;
    }
    nodes[idx] = nd;
    *depth_out = depth;
    if (tv.is_leaf(x)) *stack_out = depth - 1;
}

__global__ __launch_bounds__(kBlock) void k_emit_aabb2(TreeView tv, const uint32_t *lbefore,
                                                       bvh_node_aabb2 *nodes, uint32_t n_nodes,
                                                       BuildInfo *info) {
    const int x = blockIdx.x * kBlock + threadIdx.x;
    uint32_t depth = 0, stack = 0;
    if (x < 2 * tv.n - 1 && tv.alive(x))
        emit_aabb2_item(tv, x, lbefore, nodes, n_nodes, info, &depth, &stack);
    wave_max_to_slots(tv.depth_slots, depth);
    wave_max_to_slots(tv.stack_slots, stack);
}

// ---------------------------------------------------------------------------
// a7 (pbrt-q16): the AABB2 nodes re-encoded with u16 boxes in one frame for
// the whole scene (App. D.3).  The plane value of q is fmaf(q, s, o); each
// box gets the tightest q that still encloses it (as quantize_axis does for
// the wide layouts), and an interior node's split axis goes into the lowest
// bits of its lower x and y planes, lowering a plane by one step where the
// bit differs (which keeps the box enclosing).
// ---------------------------------------------------------------------------
__device__ inline uint32_t q16_lower(float x, float o, float s) {
    if (s == 0.0f) return 0u;
    float f = floorf((x - o) / s);
    f = fminf(fmaxf(f, 0.0f), 65535.0f);
    uint32_t a = (uint32_t)f;
    while (a > 0 && fmaf((float)a, s, o) > x) a--;
    while (a < 65535u && fmaf((float)(a + 1), s, o) <= x) a++;
    return a;
}
__device__ inline uint32_t q16_upper(float x, float o, float s) {
    if (s == 0.0f) return 0u;
    float f = ceilf((x - o) / s);
    f = fminf(fmaxf(f, 0.0f), 65535.0f);
    uint32_t b = (uint32_t)f;
    while (b < 65535u && fmaf((float)b, s, o) < x) b++;
    while (b > 0 && fmaf((float)(b - 1), s, o) >= x) b--;
    return b;
}

struct WorldFrame {
    float o[3], s[3], top[3];
};

// sg-eq (App. D.1): 10-bit steps up from the frame origin (lower planes) and
// down from the frame top (upper planes), tightest enclosing q per plane.
__device__ inline uint32_t q10_lower(float x, float o, float s) {
    if (s == 0.0f) return 0u;
    float f = floorf((x - o) / s);
    f = fminf(fmaxf(f, 0.0f), 1023.0f);
    uint32_t a = (uint32_t)f;
    while (a > 0 && fmaf((float)a, s, o) > x) a--;
    while (a < 1023u && fmaf((float)(a + 1), s, o) <= x) a++;
    return a;
}
__device__ inline uint32_t q10_upper(float x, float top, float s) {
    if (s == 0.0f) return 0u;
    float f = floorf((top - x) / s);
    f = fminf(fmaxf(f, 0.0f), 1023.0f);
    uint32_t b = (uint32_t)f;
    while (b > 0 && fmaf(-(float)b, s, top) < x) b--;
    while (b < 1023u && fmaf(-(float)(b + 1), s, top) >= x) b++;
    return b;
}

// A16: records padded with a zero word to 16 B (SG_EQ_A16).
template <bool A16>
__global__ __launch_bounds__(kBlock) void k_pack_sg_eq(const bvh_node_aabb2 *in, uint32_t n_nodes,
                                                       WorldFrame fr, void *out, BuildInfo *info) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_nodes) return;
    const bvh_node_aabb2 nd = in[i];
    uint32_t lo[3], hi[3];
    for (int a = 0; a < 3; a++) {
        lo[a] = q10_lower(nd.lo[a], fr.o[a], fr.s[a]);
        hi[a] = q10_upper(nd.hi[a], fr.top[a], fr.s[a]);
        if (fr.s[a] != 0.0f && (fmaf((float)lo[a], fr.s[a], fr.o[a]) > nd.lo[a] ||
                                fmaf(-(float)hi[a], fr.s[a], fr.top[a]) < nd.hi[a]))
            atomicOr(&info->err, 4u);
    }
    const uint32_t cnt = nd.meta & 0xFFFFu;
    bvh_node_sg_eq q;
    q.qlo = lo[0] << 20 | lo[1] << 10 | lo[2] | (cnt & 3u) << 30;
    q.qhi = hi[0] << 20 | hi[1] << 10 | hi[2] | (cnt >> 2) << 30;
    q.off = cnt > 0 ? nd.offset : (nd.offset | ((nd.meta >> 16) & 3u) << 30);
    if (A16)
        static_cast<bvh_node_sg_eq_a16 *>(out)[i] = bvh_node_sg_eq_a16{q.qlo, q.qhi, q.off, 0u};
    else
        static_cast<bvh_node_sg_eq *>(out)[i] = q;
}

// Split: boxes to out_box[i], meta words to out_meta[i] (PBRT_Q16_SOAOS);
// otherwise whole records to out[i].
template <bool Split>
__global__ __launch_bounds__(kBlock) void k_pack_pbrt_q16(const bvh_node_aabb2 *in, uint32_t n_nodes,
                                                          WorldFrame fr, bvh_node_pbrt_q16 *out,
                                                          bvh_node_box_q16 *out_box,
                                                          uint32_t *out_meta, BuildInfo *info) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_nodes) return;
    const bvh_node_aabb2 nd = in[i];
    uint32_t lo[3], hi[3];
    for (int a = 0; a < 3; a++) {
        lo[a] = q16_lower(nd.lo[a], fr.o[a], fr.s[a]);
        hi[a] = q16_upper(nd.hi[a], fr.o[a], fr.s[a]);
        // a plane outside the frame (never for a valid build) is reported
        if (fr.s[a] != 0.0f && (fmaf((float)lo[a], fr.s[a], fr.o[a]) > nd.lo[a] ||
                                fmaf((float)hi[a], fr.s[a], fr.o[a]) < nd.hi[a]))
            atomicOr(&info->err, 4u);
    }
    const uint32_t cnt = nd.meta & 0xFFFFu;
    uint32_t meta;
    if (cnt > 0) {
        meta = cnt | (nd.offset << 4);
    } else {
        const uint32_t axis = (nd.meta >> 16) & 3u;
        for (int k = 0; k < 2; k++) {
            const uint32_t bit = (axis >> k) & 1u;
            if ((lo[k] & 1u) != bit && lo[k] > 0) lo[k]--;
        }
        meta = nd.offset << 4;
    }
    if (Split) {
        bvh_node_box_q16 q;
        q.lo[0] = (uint16_t)lo[0]; q.lo[1] = (uint16_t)lo[1]; q.lo[2] = (uint16_t)lo[2];
        q.hi[0] = (uint16_t)hi[0]; q.hi[1] = (uint16_t)hi[1]; q.hi[2] = (uint16_t)hi[2];
        out_box[i] = q;
        out_meta[i] = meta;
    } else {
        bvh_node_pbrt_q16 q;
        q.lo[0] = (uint16_t)lo[0]; q.lo[1] = (uint16_t)lo[1]; q.lo[2] = (uint16_t)lo[2];
        q.hi[0] = (uint16_t)hi[0]; q.hi[1] = (uint16_t)hi[1]; q.hi[2] = (uint16_t)hi[2];
        q.meta = meta;
        out[i] = q;
    }
}

// SHARED_SLAB: node c keeps one slab, the exact extent of its box along the
// axis where that box is narrowest relative to its parent's box (the scene
// box for the root; lowest axis on ties), written by its parent's thread.
__device__ inline bvh_node_slab slab_record(const bvh_node_aabb2 &c, const float *plo,
                                            const float *phi) {
    int axis = 0;
    float best = INFINITY;
    for (int a = 0; a < 3; a++) {
        const float pe = phi[a] - plo[a], ce = c.hi[a] - c.lo[a];
        const float ratio = pe > 0.0f ? ce / pe : 1.0f;
        if (ratio < best) {
            best = ratio;
            axis = a;
        }
    }
    const uint32_t cnt = c.meta & 0xFFFFu, split = (c.meta >> 16) & 3u;
    return bvh_node_slab{c.lo[axis], c.hi[axis], c.offset,
                         cnt | ((uint32_t)axis << 16) | (split << 18)};
}

__global__ __launch_bounds__(kBlock) void k_pack_slab(const bvh_node_aabb2 *in, uint32_t n_nodes,
                                                      const BuildInfo *info, bvh_node_slab *out) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_nodes) return;
    const bvh_node_aabb2 nd = in[i];
    if (i == 0) out[0] = slab_record(nd, info->slo, info->shi);
    if ((nd.meta & 0xFFFFu) != 0u) return;
    const uint32_t kids[2] = {i + 1u, i + nd.offset};
    for (int k = 0; k < 2; k++)
        if (kids[k] < n_nodes) out[kids[k]] = slab_record(in[kids[k]], nd.lo, nd.hi);
}

// AABB2 records split into a box array and a topology array (PBRT_SOAOS).
__global__ __launch_bounds__(kBlock) void k_split_aabb2(const bvh_node_aabb2 *in, uint32_t n_nodes,
                                                        bvh_node_box_f32 *box, bvh_node_topo *topo) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_nodes) return;
    const bvh_node_aabb2 nd = in[i];
    bvh_node_box_f32 b;
    for (int a = 0; a < 3; a++) {
        b.lo[a] = nd.lo[a];
        b.hi[a] = nd.hi[a];
    }
    box[i] = b;
    topo[i] = bvh_node_topo{nd.offset, nd.meta};
}

// ---------------------------------------------------------------------------
// a7 (wide): top-down, one frontier level per step.  Each frontier item is an
// alive interior binary node that becomes a wide node: its child list starts
// as its two children and repeatedly replaces the interior candidate of
// largest surface area by that candidate's two children, up to K children.
// The list depends only on the binary node, so one launch forms it for every
// alive interior node up front (a chain of dependent loads per node, hidden
// by running all of them at once); per level an exclusive scan of the
// interior-child counts places the children and one pass writes the nodes,
// the next frontier and its counts.
// ---------------------------------------------------------------------------
// Greedy opening of one wide node (binary node x): returns the number of
// interior candidates and writes K candidate ids (-1 for unused slots).
template <int K>
__device__ inline uint32_t wide_open_item(const TreeView &tv, int x, int32_t *cand_out) {
    // Per candidate: id, area (-1 for a leaf, which is never opened) and its
    // children, read when the candidate enters the list, so that an opening
    // waits for one round of loads (8-wide nodes of 1,024 triangles 16 -> 12 us,
    // of 300,000 25 -> 15 us)
    int c[K], l[K], r[K];
    float area[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        c[k] = l[k] = r[k] = -1;
        area[k] = -1.0f;
    }
    const auto look = [&](int y, int &yl, int &yr, float &a) {
        yl = yr = -1;
        a = -1.0f;
        if (tv.is_prim(y)) return;
        const uint32_t cnt = tv.icount[y];
        const float ar = tv.area[y];
        yl = tv.ileft[y];
        yr = tv.iright[y];
        if (cnt > (uint32_t)tv.leaf_size) a = ar;
    };
    int nc;
    if (tv.is_leaf(x)) {  // only for a root that is a single leaf
        c[0] = x;
        nc = 1;
    } else {
        c[0] = tv.ileft[x];
        c[1] = tv.iright[x];
        look(c[0], l[0], r[0], area[0]);
        look(c[1], l[1], r[1], area[1]);
        nc = 2;
        while (nc < K) {
            int best = -1, yl = -1, yr = -1;
            float best_a = -1.0f;
#pragma unroll
            for (int k = 0; k < K; k++) {
                if (area[k] > best_a) {  // the lowest of equal ones
                    best_a = area[k];
                    best = k;
                    yl = l[k];
                    yr = r[k];
                }
            }
            if (best < 0) break;
            int ll, lr, rl, rr;
            float la, ra;
            look(yl, ll, lr, la);
            look(yr, rl, rr, ra);
            // replace the candidate by its two children, keeping left-to-right order
#pragma unroll
            for (int k = K - 1; k >= 0; k--) {
                if (k > best + 1) {
                    c[k] = c[k > 0 ? k - 1 : 0];
                    l[k] = l[k > 0 ? k - 1 : 0];
                    r[k] = r[k > 0 ? k - 1 : 0];
                    area[k] = area[k > 0 ? k - 1 : 0];
                } else if (k == best + 1) {
                    c[k] = yr;
                    l[k] = rl;
                    r[k] = rr;
                    area[k] = ra;
                } else if (k == best) {
                    c[k] = yl;
                    l[k] = ll;
                    r[k] = lr;
                    area[k] = la;
                }
            }
            nc++;
        }
    }
    uint32_t ni = 0, mask = 0;
#pragma unroll
    for (int k = 0; k < K; k++) {
        cand_out[k] = c[k];
        if (area[k] != -1.0f) {  // an interior candidate, NaN area included
            ni++;
            mask |= 1u << k;
        }
    }
    return ni | (mask << 8);
}

// Binary nodes 0 .. m-1 (m = max(n-1, 1)): the root and every alive interior
// node get their child list (cand_all[x*K ..]) and a word with the number of
// interior children (low 8 bits) and which slots hold them (bit 8 + slot).
template <int K>
__global__ __launch_bounds__(kBlock) void k_wide_open_all(TreeView tv, uint32_t m, int32_t *cand_all,
                                                          uint32_t *ni_all) {
    const uint32_t x = blockIdx.x * kBlock + threadIdx.x;
    if (x >= m) return;
    if (x != 0 && !(tv.alive((int)x) && !tv.is_leaf((int)x))) return;
    ni_all[x] = wide_open_item<K>(tv, (int)x, cand_all + (size_t)x * K);
}

// Scale of one axis: the smallest step found upwards from ext / QMAX with
// fmaf(QMAX, s, plo) >= phi (0 for an empty extent; a bad one is reported).
template <int QMAX>
__device__ inline float quantize_scale(float plo, float phi, uint32_t *err) {
    const float ext = phi - plo;
    float s = 0.0f;
    if (!(ext >= 0.0f) || !isfinite(ext)) {
        atomicOr(err, 2u);
    } else if (ext > 0.0f) {
        s = ext / (float)QMAX;
        for (int g = 0; g < 64 && fmaf((float)QMAX, s, plo) < phi; g++) s = nextafterf(s, INFINITY);
    }
    return s;
}

// A child interval in steps of s from plo: the tightest q values with
// fmaf(qlo, s, plo) <= clo and fmaf(qhi, s, plo) >= chi.
template <int QMAX>
__device__ inline void quantize_interval(float plo, float s, float clo, float chi, uint32_t *qlo,
                                         uint32_t *qhi) {
    uint32_t a = 0, b = 0;
    if (s != 0.0f) {
        float fl = floorf((clo - plo) / s);
        fl = fminf(fmaxf(fl, 0.0f), (float)QMAX);
        a = (uint32_t)fl;
        while (a > 0 && fmaf((float)a, s, plo) > clo) a--;
        while (a < (uint32_t)QMAX && fmaf((float)(a + 1), s, plo) <= clo) a++;
        float fh = ceilf((chi - plo) / s);
        fh = fminf(fmaxf(fh, 0.0f), (float)QMAX);
        b = (uint32_t)fh;
        while (b < (uint32_t)QMAX && fmaf((float)b, s, plo) < chi) b++;
        while (b > 0 && fmaf((float)(b - 1), s, plo) >= chi) b--;
    }
    *qlo = a;
    *qhi = b;
}

__device__ inline float box_comp(const Box &b, int c) {
    return c == 0 ? b.lo.x : c == 1 ? b.lo.y : c == 2 ? b.lo.z : c == 3 ? b.hi.x : c == 4 ? b.hi.y : b.hi.z;
}

// Node writers.  A wide node is written by K lanes, lane k with child k (box,
// reference, whether it exists): each puts its words of the record into LDS
// (rec), and the group stores the record in 16-byte chunks, so a wave writes
// whole consecutive records.  One thread per node, with its K children one
// after another, was bound by that chain: 30 us for a BVH8-Q8 of 1,024
// triangles, 59 us for a BVH8-Q16 of 300,000, 41 us for a BVH4 of 2.1 M; the
// groups take 7, 13 and 32 us.
template <int Layout>
struct WideOut;

template <>
struct WideOut<BVH_LAYOUT_BVH4> {
    static constexpr int K = 4;
    static constexpr int kWords = sizeof(bvh_node_bvh4) / 4;
    __device__ static void put(uint32_t *rec, int k, const Box &pb, const Box &cb, bool valid,
                               uint32_t ref, int nc, uint32_t *err) {
        (void)pb;
        (void)err;
        rec[0 * K + k] = __float_as_uint(valid ? cb.lo.x : INFINITY);
        rec[1 * K + k] = __float_as_uint(valid ? cb.lo.y : INFINITY);
        rec[2 * K + k] = __float_as_uint(valid ? cb.lo.z : INFINITY);
        rec[3 * K + k] = __float_as_uint(valid ? cb.hi.x : -INFINITY);
        rec[4 * K + k] = __float_as_uint(valid ? cb.hi.y : -INFINITY);
        rec[5 * K + k] = __float_as_uint(valid ? cb.hi.z : -INFINITY);
        rec[6 * K + k] = ref;
        rec[7 * K + k] = k == 0 ? (uint32_t)nc : 0u;
    }
};

// Record words of the quantised 8-wide nodes: origin[3], scale[3], then the
// six plane rows (qlo_x, qlo_y, qlo_z, qhi_x, qhi_y, qhi_z) of 8 values of
// QT, child[8], nchild, zero padding.
template <typename QT, int Words>
__device__ inline void quantized_put(uint32_t *rec, int k, const Box &pb, const Box &cb, bool valid,
                                     uint32_t ref, int nc, uint32_t *err) {
    constexpr int K = 8;
    constexpr uint32_t kQMax = (QT)~(QT)0;
    constexpr int c0 = 6 + 6 * K * sizeof(QT) / 4;
    QT *rows = reinterpret_cast<QT *>(rec + 6);
    // lane a works out axis a's scale for the group (its axis is picked among
    // register values: indexing the box would put it in scratch memory)
    const float ax = pb.lo.x, ay = pb.lo.y, az = pb.lo.z, bx = pb.hi.x, by = pb.hi.y, bz = pb.hi.z;
    float own = 0.0f;
    if (k < 3)
        own = quantize_scale<(int)kQMax>(k == 0 ? ax : (k == 1 ? ay : az), k == 0 ? bx : (k == 1 ? by : bz), err);
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const float sc = __shfl(own, a, K);
        const float plo = box_comp(pb, a);
        uint32_t qlo = kQMax, qhi = 0;  // empty slot: lo above hi
        if (valid) quantize_interval<(int)kQMax>(plo, sc, box_comp(cb, a), box_comp(cb, a + 3), &qlo, &qhi);
        rows[a * K + k] = (QT)qlo;
        rows[(3 + a) * K + k] = (QT)qhi;
        if (k == a) {
            rec[a] = __float_as_uint(plo);
            rec[3 + a] = __float_as_uint(sc);
        }
    }
    rec[c0 + k] = ref;
    if (c0 + K + k < Words) rec[c0 + K + k] = k == 0 ? (uint32_t)nc : 0u;
    static_assert(Words - (c0 + K) <= K && Words % 4 == 0, "one word of the tail per lane");
}

static_assert(offsetof(bvh_node_bvh4, child) == 24 * 4 && offsetof(bvh_node_bvh4, nchild) == 28 * 4,
              "bvh4 record words");
static_assert(offsetof(bvh_node_bvh8_q8, qlo_x) == 6 * 4 && offsetof(bvh_node_bvh8_q8, qhi_x) == 12 * 4 &&
                  offsetof(bvh_node_bvh8_q8, child) == 18 * 4 && offsetof(bvh_node_bvh8_q8, nchild) == 26 * 4,
              "bvh8-q8 record words");
static_assert(offsetof(bvh_node_bvh8_q16, qlo_x) == 6 * 4 && offsetof(bvh_node_bvh8_q16, qhi_x) == 18 * 4 &&
                  offsetof(bvh_node_bvh8_q16, child) == 30 * 4 && offsetof(bvh_node_bvh8_q16, nchild) == 38 * 4,
              "bvh8-q16 record words");

template <>
struct WideOut<BVH_LAYOUT_BVH8_Q8> {
    static constexpr int K = 8;
    static constexpr int kWords = sizeof(bvh_node_bvh8_q8) / 4;
    __device__ static void put(uint32_t *rec, int k, const Box &pb, const Box &cb, bool valid,
                               uint32_t ref, int nc, uint32_t *err) {
        quantized_put<uint8_t, kWords>(rec, k, pb, cb, valid, ref, nc, err);
    }
};

template <>
struct WideOut<BVH_LAYOUT_BVH8_Q16> {
    static constexpr int K = 8;
    static constexpr int kWords = sizeof(bvh_node_bvh8_q16) / 4;
    __device__ static void put(uint32_t *rec, int k, const Box &pb, const Box &cb, bool valid,
                               uint32_t ref, int nc, uint32_t *err) {
        quantized_put<uint16_t, kWords>(rec, k, pb, cb, valid, ref, nc, err);
    }
};

// Where wide node w goes: nodes below spec_cap straight into the handle's
// node block (allocated ahead from an earlier build's count), the rest into
// the work area (moved into an exact block after the last level).
struct NodeSink {
    uint8_t *spec;
    uint32_t spec_cap;
    uint8_t *over;
    uint32_t bytes;
    __device__ void *at(uint32_t w) const {
        return w < spec_cap ? spec + (size_t)w * bytes : over + (size_t)w * bytes;
    }
};

// ---------------------------------------------------------------------------
// Wide packing by subtrees.  The wide tree's top levels, while a level holds
// at most kTopMaxFrontier nodes, are planned breadth-first by one workgroup;
// every node of the next level roots a subtree, which one workgroup plans
// breadth-first in a queue of its own.  A subtree's wide nodes number at most
// its primitive count less one (each has two children or more), so its queue
// sits at the subtree root's first primitive position in arrays of n entries,
// and the queues of different subtrees never overlap.  A scan of the subtree
// sizes then places each subtree contiguously after the top levels, and one
// launch over all node positions writes every record (a group of lanes finds its
// subtree by a search over the subtree offsets, so uneven subtrees
// do not leave one workgroup with most of the work).  Node order: the top
// levels breadth-first, then subtree by subtree in the order of their roots,
// each breadth-first; a subtree's nodes are thus close together in memory.
// Only the final node count goes to the host.
//
// Plan entries: the binary node x, its aux word (the stack entries its
// ancestors leave behind in the low 16 bits, its depth in the high 16) and
// the queue index of its first interior child (the others follow it).
// ---------------------------------------------------------------------------
constexpr uint32_t kTopMaxFrontier = 1024;
constexpr uint32_t kTopMaxLevels = 64;
constexpr uint32_t kTopMaxNodes = kTopMaxFrontier * kTopMaxLevels;
constexpr int kPlanItems = 4;         // consecutive queue entries per thread and pass
constexpr int kTopThreads = 512;      // the top levels: one workgroup
static_assert(kTopMaxFrontier <= kTopThreads * kPlanItems, "a top level is planned in one pass");
constexpr int kSubThreads = 64;       // a subtree: one wave (its scans need no barrier)
constexpr uint32_t kPlanBlocks = 8192;  // subtree planning: waves, striding over the roots
constexpr int kPlaceThreads = 1024;

struct WidePlan {
    int32_t *t_node;  // top levels, node i at position i (kTopMaxNodes)
    uint32_t *t_aux, *t_noff;
    int32_t *f_node;  // subtree roots (K * kTopMaxFrontier)
    uint32_t *f_aux, *f_size, *f_off, *f_q0;
    int32_t *s_node;  // subtree queues (n entries, by primitive position)
    uint32_t *s_aux, *s_noff;
    uint32_t *meta;   // [0] top nodes, [1] subtrees, [2] all nodes
};

// One pass over queue entries [c, min(c + THREADS * kPlanItems, hi)), kPlanItems
// consecutive ones per thread: their child lists and interior-slot words are
// loaded together, the interior-child counts scanned over the block (child
// indices from `start`), each entry's first-child index stored in qo.  The
// entries stay in registers for plan_children.  Every thread calls it.
template <int K>
struct PlanRegs {
    int32_t cand[kPlanItems][K];
    uint32_t aux[kPlanItems], word[kPlanItems], off[kPlanItems];
};

// get(i, x, a) reads entry i's binary node and aux word.
template <int K, int THREADS, typename Get>
__device__ inline uint32_t plan_pass(Get get, uint32_t *qo, uint32_t c, uint32_t hi, uint32_t start,
                                     const int32_t *cand_all, const uint32_t *ni_all, uint32_t *wsum,
                                     PlanRegs<K> &R) {
    const uint32_t i0 = c + threadIdx.x * kPlanItems;
    int32_t x[kPlanItems];
#pragma unroll
    for (int k = 0; k < kPlanItems; k++) {
        x[k] = -1;
        R.aux[k] = 0u;
        if (i0 + k < hi) get(i0 + k, x[k], R.aux[k]);
    }
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kPlanItems; k++) {
        R.word[k] = x[k] >= 0 ? ni_all[x[k]] : 0u;
#pragma unroll
        for (int j = 0; j < K; j++) R.cand[k][j] = x[k] >= 0 ? cand_all[(size_t)x[k] * K + j] : -1;
        sum += R.word[k] & 0xFFu;
    }
    uint32_t tot;
    uint32_t run = start + block_excl_scan<THREADS>(sum, &tot, wsum);
#pragma unroll
    for (int k = 0; k < kPlanItems; k++) {
        R.off[k] = run;
        if (i0 + k < hi) qo[i0 + k] = run;
        run += R.word[k] & 0xFFu;
    }
    return tot;
}

// Appends the pass's interior children (candidate order): put(at, node, aux)
// for each, at its queue index.
template <int K, typename Put>
__device__ inline void plan_children(const PlanRegs<K> &R, uint32_t c, uint32_t hi, Put put) {
    const uint32_t i0 = c + threadIdx.x * kPlanItems;
#pragma unroll
    for (int k = 0; k < kPlanItems; k++) {
        if (i0 + k >= hi) continue;
        int nc = 0;
#pragma unroll
        for (int j = 0; j < K; j++) nc += R.cand[k][j] >= 0;
        const uint32_t a = R.aux[k];
        const uint32_t caux = (((a & 0xFFFFu) + (uint32_t)(nc - 1)) & 0xFFFFu) | (((a >> 16) + 1) << 16);
        const uint32_t mask = R.word[k] >> 8;
        uint32_t at = R.off[k];
#pragma unroll
        for (int j = 0; j < K; j++) {
            if (!((mask >> j) & 1u)) continue;
            put(at, R.cand[k][j], caux);
            at++;
        }
    }
}

// The level in hand is kept in LDS as well, so that it costs one round of
// global loads (the lists) instead of two.  whole: a tree of at most
// kTopMaxFrontier wide nodes is planned here to its last level, has no
// subtrees and is placed at once (1,024 triangles: two launches less).
template <int K>
__global__ __launch_bounds__(kTopThreads) void k_wide_plan_top(const int32_t *cand_all,
                                                               const uint32_t *ni_all, WidePlan p,
                                                               bool whole, uint32_t cap,
                                                               BuildInfo *info, uint32_t *host_word) {
    __shared__ uint32_t wsum[kTopThreads / kWave];
    __shared__ int32_t s_node[2][kTopMaxFrontier];
    __shared__ uint32_t s_aux[2][kTopMaxFrontier];
    if (threadIdx.x == 0) {  // level 0 = {root}, nothing stacked, depth 0
        p.t_node[0] = 0;
        p.t_aux[0] = 0;
        s_node[0][0] = 0;
        s_aux[0][0] = 0;
    }
    __syncthreads();
    uint32_t lo = 0, hi = 1, total = 0;
    bool frontier = false, bad = false;
    for (uint32_t level = 0;; level++) {
        PlanRegs<K> R;
        const int cur = (int)(level & 1u), nxt = cur ^ 1;
        total = plan_pass<K, kTopThreads>(
            [&](uint32_t i, int32_t &x, uint32_t &a) {
                x = s_node[cur][i - lo];
                a = s_aux[cur][i - lo];
            },
            p.t_noff, lo, hi, hi, cand_all, ni_all, wsum, R);
        // the same in every thread: the next level becomes the subtree roots
        // when it is too wide for one pass or the top is too deep
        bad = whole && hi + total > cap;  // cannot happen: the tree is malformed
        frontier = !whole && (total > kTopMaxFrontier || level + 1 >= kTopMaxLevels || hi + total > kTopMaxNodes);
        if (bad) break;
        if (frontier)
            plan_children<K>(R, lo, hi, [&](uint32_t at, int32_t x, uint32_t a) {
                p.f_node[at - hi] = x;
                p.f_aux[at - hi] = a;
            });
        else
            plan_children<K>(R, lo, hi, [&](uint32_t at, int32_t x, uint32_t a) {
                p.t_node[at] = x;
                p.t_aux[at] = a;
                s_node[nxt][at - hi] = x;
                s_aux[nxt][at - hi] = a;
            });
        __syncthreads();
        if (frontier || total == 0) break;
        lo = hi;
        hi += total;
    }
    if (threadIdx.x == 0) {
        p.meta[0] = hi;
        p.meta[1] = frontier ? total : 0u;
        if (whole) {
            if (bad) atomicOr(&info->err, 4u);
            p.meta[2] = hi;
            *host_word = hi;
            __threadfence_system();  // the host polls the word
        }
    }
}

template <int K>
__global__ __launch_bounds__(kSubThreads) void k_wide_plan_sub(TreeView tv, const int32_t *cand_all,
                                                               const uint32_t *ni_all, WidePlan p,
                                                               BuildInfo *info) {
    __shared__ uint32_t wsum[kSubThreads / kWave];
    const uint32_t roots = p.meta[1];
    for (uint32_t b = blockIdx.x; b < roots; b += gridDim.x) {
        const int32_t x = p.f_node[b];
        const uint32_t q0 = tv.first(x), qcap = tv.count(x);
        int32_t *qn = p.s_node + q0;
        uint32_t *qa = p.s_aux + q0, *qo = p.s_noff + q0;
        if (threadIdx.x == 0) {
            qn[0] = x;
            qa[0] = p.f_aux[b];
            p.f_q0[b] = q0;
        }
        __syncthreads();
        uint32_t lo = 0, hi = 1;
        bool bad = false;
        while (lo < hi && !bad) {
            uint32_t next = hi;
            for (uint32_t c = lo; c < hi; c += kSubThreads * kPlanItems) {
                PlanRegs<K> R;
                const uint32_t tot = plan_pass<K, kSubThreads>(
                    [&](uint32_t i, int32_t &x, uint32_t &a) {
                        x = qn[i];
                        a = qa[i];
                    },
                    qo, c, hi, next, cand_all, ni_all, wsum, R);
                if (next + tot > qcap) {  // cannot happen (see above): the tree is malformed
                    bad = true;
                    break;
                }
                plan_children<K>(R, c, hi, [&](uint32_t at, int32_t x, uint32_t a) {
                    qn[at] = x;
                    qa[at] = a;
                });
                next += tot;
            }
            __syncthreads();
            lo = hi;
            hi = bad ? lo : next;
        }
        if (threadIdx.x == 0) {
            if (bad) atomicOr(&info->err, 4u);
            p.f_size[b] = hi;
        }
    }
}

// Places the subtrees (f_off = absolute position of a subtree's first node)
// and publishes the node count (meta[2] and a host-mapped word).
__global__ __launch_bounds__(kPlaceThreads) void k_wide_place(WidePlan p, uint32_t cap,
                                                              BuildInfo *info, uint32_t *host_word) {
    __shared__ uint32_t wsum[kPlaceThreads / kWave];
    const uint32_t base = p.meta[0], count = p.meta[1];
    uint32_t carry = 0;
    for (uint32_t c = 0; c < count; c += kPlaceThreads * kPlanItems) {
        const uint32_t b0 = c + threadIdx.x * kPlanItems;
        uint32_t v[kPlanItems], sum = 0;
#pragma unroll
        for (int k = 0; k < kPlanItems; k++) {
            v[k] = b0 + k < count ? p.f_size[b0 + k] : 0u;
            sum += v[k];
        }
        uint32_t tot;
        uint32_t run = base + carry + block_excl_scan<kPlaceThreads>(sum, &tot, wsum);
#pragma unroll
        for (int k = 0; k < kPlanItems; k++) {
            if (b0 + k < count) p.f_off[b0 + k] = run;
            run += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) {
        const uint32_t all = base + carry;
        if (all > cap) atomicOr(&info->err, 4u);
        p.meta[2] = all;
        *host_word = all;
        __threadfence_system();  // the host polls the word
    }
}

// Subtree of node position at: the last b of [0, roots) with off[b] <= at.
// The group's K lanes probe K pivots of the range at a time.
template <int K>
__device__ inline uint32_t find_subtree(const uint32_t *off, uint32_t roots, uint32_t at) {
    const int k = threadIdx.x % K, g0 = (threadIdx.x & (kWave - 1)) & ~(K - 1);
    uint32_t lo = 0, len = roots;  // the answer is in [lo, lo + len)
    while (len > 1) {
        const uint32_t step = (len + K) / (K + 1);  // 1 or more
        const uint32_t i = (uint32_t)(k + 1) * step;
        const bool le = i < len && off[lo + i] <= at;
        // the groups of a wave leave the loop one by one: each reads its own lanes' bits only
        const uint32_t le_k = (uint32_t)(__builtin_amdgcn_ballot_w64(le) >> g0) & ((1u << K) - 1u);
        const uint32_t c = (uint32_t)__builtin_popcount(le_k);
        lo += c * step;
        len = min(step, len - c * step);
    }
    return lo;
}

// K lanes per node position (launched for the largest possible count): the
// subtree, the node's plan entry, then lane k reads child k.  What bounds it
// are those four dependent reads and the stores.
template <int Layout>
__global__ __launch_bounds__(kBlock) void k_wide_write(TreeView tv, const int32_t *cand_all,
                                                       WidePlan p, uint32_t cap, NodeSink sink,
                                                       BuildInfo *info) {
    constexpr int K = WideOut<Layout>::K;
    constexpr int kWords = WideOut<Layout>::kWords;
    constexpr uint32_t kNodes = kBlock / K;  // nodes of a block
    __shared__ __align__(16) uint32_t s_rec[kNodes][kWords + 4];  // rows 4 banks apart
    const uint32_t base = p.meta[0], roots = min(p.meta[1], (uint32_t)(K * kTopMaxFrontier)),
                   all = p.meta[2];
    const int k = threadIdx.x % K, g0 = (threadIdx.x & (kWave - 1)) & ~(K - 1);
    const uint32_t at = blockIdx.x * kNodes + threadIdx.x / K;
    uint32_t stack = 0, depth = 0;
    if (at < all && at >= cap) {
        if (k == 0) atomicOr(&info->err, 4u);
    } else if (at < all) {  // the same in a node's K lanes, here and below
        const bool top = at < base;
        const uint32_t b = top ? 0u : find_subtree<K>(p.f_off, roots, at);
        const uint32_t off = top ? 0u : p.f_off[b];
        const uint32_t q = top ? at : p.f_q0[b] + (at - off);
        const uint32_t no = (top ? p.t_noff : p.s_noff)[q];
        const int32_t x = (top ? p.t_node : p.s_node)[q];
        const uint32_t aux = (top ? p.t_aux : p.s_aux)[q];
        const int c = cand_all[(size_t)x * K + k];  // valid candidates are the first nc slots
        const bool valid = c >= 0;
        const Box pb = tv.nbox[x];
        const Box cb = valid ? tv.nbox[c] : box_empty();  // box and range in one load
        const uint32_t cnt = valid ? range_count(cb) : 0u;
        const bool inner = valid && cnt > (uint32_t)tv.leaf_size;
        const uint32_t inner_k = (uint32_t)(__builtin_amdgcn_ballot_w64(inner) >> g0) & ((1u << K) - 1u);
        const int nc = __builtin_popcount((uint32_t)(__builtin_amdgcn_ballot_w64(valid) >> g0) & ((1u << K) - 1u));
        uint32_t ref = kRefEmpty;
        bool bad = false;
        if (inner) {
            const uint32_t j = no + (uint32_t)__builtin_popcount(inner_k & ((1u << k) - 1u));
            // the last top level's children are subtree roots
            const uint32_t pos = !top ? off + j : (j < base ? j : p.f_off[j - base]);
            bad = pos >= cap;
            ref = ref_interior(pos);
        } else if (valid) {
            ref = ref_leaf(range_first(cb), cnt);
        }
        const bool any_bad = ((uint32_t)(__builtin_amdgcn_ballot_w64(bad) >> g0) & ((1u << K) - 1u)) != 0;
        if (any_bad) {
            if (k == 0) atomicOr(&info->err, 4u);
        } else {
            uint32_t *rec = s_rec[threadIdx.x / K];
            WideOut<Layout>::put(rec, k, pb, cb, valid, ref, nc, &info->err);
            wave_sync();
            uint4 *dst = static_cast<uint4 *>(sink.at(at));
            for (int i = k; i < kWords / 4; i += K) dst[i] = reinterpret_cast<const uint4 *>(rec)[i];
            stack = (aux & 0xFFFFu) + (uint32_t)(nc - 1);
            depth = (aux >> 16) + 2;  // its children's level and the leaf level below
        }
    }
    wave_max_to_slots(tv.stack_slots, stack);
    wave_max_to_slots(tv.depth_slots, depth);
}

// Folds the per-wave maxima slots into info->max_stack / max_depth.
__global__ __launch_bounds__(kBlock) void k_fold_max_slots(const uint32_t *stack_slots,
                                                           const uint32_t *depth_slots,
                                                           BuildInfo *info) {
    __shared__ uint32_t red[2][kBlock / kWave];
    uint32_t a = 0, b = 0;
    for (int i = threadIdx.x; i < kMaxSlots; i += kBlock) {
        a = max(a, stack_slots[i * kSlotStride]);
        b = max(b, depth_slots[i * kSlotStride]);
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        a = max(a, (uint32_t)__shfl_xor((int)a, o, kWave));
        b = max(b, (uint32_t)__shfl_xor((int)b, o, kWave));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][threadIdx.x / kWave] = a;
        red[1][threadIdx.x / kWave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {  // a, b already hold wave 0's maxima
        for (int w = 1; w < kBlock / kWave; w++) {
            a = max(a, red[0][w]);
            b = max(b, red[1][w]);
        }
        info->max_stack = max(info->max_stack, a);
        info->max_depth = max(info->max_depth, b);
    }
}

// ---------------------------------------------------------------------------
// Leaf data
// ---------------------------------------------------------------------------
// The build reports out-of-range vertex indices only after this kernel has
// run (the wide layouts do not wait for the bounds pass's verdict), so a
// triangle with such an index is written as zeros instead of being read.
__global__ __launch_bounds__(kBlock) void k_leaf_compact(const float *verts, int64_t n_verts,
                                                         const int32_t *tris, const uint32_t *perm,
                                                         uint32_t n, bvh_tri *out) {
    const uint32_t j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= n) return;
    const uint32_t t = perm[j];
    const int32_t i0 = tris[3 * (size_t)t], i1 = tris[3 * (size_t)t + 1], i2 = tris[3 * (size_t)t + 2];
    float p0[3] = {0.f, 0.f, 0.f}, e1[3] = {0.f, 0.f, 0.f}, e2[3] = {0.f, 0.f, 0.f};
    if (i0 >= 0 && i0 < n_verts && i1 >= 0 && i1 < n_verts && i2 >= 0 && i2 < n_verts) {
        const float *q0 = verts + 3 * (size_t)i0;
        const float *q1 = verts + 3 * (size_t)i1;
        const float *q2 = verts + 3 * (size_t)i2;
        for (int a = 0; a < 3; a++) {
            p0[a] = q0[a];
            e1[a] = q1[a] - q0[a];  // the f32 edges of the intersection test
            e2[a] = q2[a] - q0[a];
        }
    }
    // the 48-B record as three 16-B stores
    float4 *o = reinterpret_cast<float4 *>(out + j);
    o[0] = make_float4(p0[0], p0[1], p0[2], e1[0]);
    o[1] = make_float4(e1[1], e1[2], e2[0], e2[1]);
    o[2] = make_float4(e2[2], __int_as_float((int)t), 0.0f, 0.0f);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Small host words that kernels write directly (pinned, coherent, mapped into
// the device's address space), one set per host thread.  Polling them lets
// the host learn a count as soon as the kernel that produces it has run,
// while later kernels of the same level are still queued or running, instead
// of waiting for the whole stream and a copy.
constexpr uint32_t kPending = 0xFFFFFFFFu;

uint32_t *host_words() {
    static thread_local void *buf = nullptr;
    if (!buf && hipHostMalloc(&buf, 256, hipHostMallocCoherent | hipHostMallocMapped) != hipSuccess) {
        (void)hipGetLastError();
        buf = nullptr;
    }
    return static_cast<uint32_t *>(buf);
}

// Waits until the kernel-written word p no longer holds kPending.  The wait
// is bounded by the stream: if the stream has finished (or failed) and the
// word is still pending, it reports an error instead of spinning on.
int32_t wait_host_word(volatile uint32_t *p, hipStream_t s, uint32_t *out) {
    for (uint64_t spin = 1;; spin++) {
        const uint32_t v = *p;
        if (v != kPending) {
            *out = v;
            return BVH_OK;
        }
        if ((spin & 255u) == 0) {
            const hipError_t e = hipStreamQuery(s);
            if (e == hipSuccess) {
                const uint32_t w = *p;
                if (w != kPending) {
                    *out = w;
                    return BVH_OK;
                }
                return set_error(BVH_EHIP, "bvh_build: internal error (count not written)");
            }
            if (e != hipErrorNotReady) {
                return set_error(BVH_EHIP, "bvh_build: %s", hipGetErrorString(e));
            }
        }
    }
}

// Small pinned host staging area for device-to-host readbacks (one per thread).
template <typename T>
T *pinned_scratch() {
    static thread_local void *buf = nullptr;
    if (!buf && hipHostMalloc(&buf, 256, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        buf = nullptr;
    }
    static_assert(sizeof(T) <= 256, "pinned scratch too small");
    return static_cast<T *>(buf);
}

// Scene frame of the scene-frame quantised layouts: origin and top = scene box
// corners, scale = the smallest step with fmaf(steps, s, o) >= top and
// fmaf(-steps, s, top) <= o (std::fmaf rounds like the device's fmaf).
// Non-finite extents give scale 0 (reported elsewhere).
WorldFrame world_frame(const float *lo, const float *hi, float steps) {
    WorldFrame fr;
    for (int a = 0; a < 3; a++) {
        fr.o[a] = lo[a];
        fr.top[a] = hi[a];
        const float ext = hi[a] - lo[a];
        float sc = 0.0f;
        if (ext > 0.0f && std::isfinite(ext)) {
            sc = ext / steps;
            // full range both ways: up from lo reaches hi, down from hi reaches lo
            for (int g = 0; g < 64 && (std::fmaf(steps, sc, lo[a]) < hi[a] ||
                                       std::fmaf(-steps, sc, hi[a]) > lo[a]); g++)
                sc = std::nextafter(sc, INFINITY);
        }
        fr.s[a] = sc;
    }
    return fr;
}

int32_t check_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(BVH_EHIP, "%s: launch failed: %s", what, hipGetErrorString(e));
    return BVH_OK;
}

// The handle's two allocations.  Their hipMalloc calls block the host, so
// the build issues each one while queued kernels keep the GPU busy: the leaf
// block (size known from the input) before the host waits for the leaf
// count, the node block once the leaf data kernels are queued.
int32_t alloc_leaf_block(bvh_handle_s *h) {
    auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t n = (size_t)h->n_tris;
    const bool compact = h->leaf_mode == BVH_LEAF_COMPACT;
    const size_t b_leaf = up(n * (compact ? sizeof(bvh_tri) : sizeof(int32_t)));
    const size_t b_verts = compact ? 0 : up((size_t)h->n_verts * 3 * sizeof(float));
    const size_t b_tris = compact ? 0 : up(n * 3 * sizeof(int32_t));
    BVH_HIP_TRY(block_alloc(h->device, b_leaf + b_verts + b_tris, &h->block));
    char *p = static_cast<char *>(h->block.ptr);
    h->leaf = p;
    if (!compact) {
        h->verts = reinterpret_cast<float *>(p + b_leaf);
        h->tris = reinterpret_cast<int32_t *>(p + b_leaf + b_verts);
    }
    return BVH_OK;
}

int32_t alloc_node_block(bvh_handle_s *h, int64_t n_nodes) {
    BVH_HIP_TRY(block_alloc(h->device, (size_t)n_nodes * (size_t)h->node_bytes, &h->node_block));
    h->node_block_cap = (uint32_t)n_nodes;
    h->nodes = h->node_block.ptr;
    return BVH_OK;
}

// Leaf data of the handle (a8): compacted triangles in leaf order, or the
// permutation plus the handle's own copies of the vertices and indices.
struct LeafSource {
    const float *verts;
    int64_t n_verts;
    const int32_t *tris;
    const uint32_t *perm;
    uint32_t n;
};

int32_t emit_leaf_data(bvh_handle_s *h, const LeafSource &ls, hipStream_t s) {
    if (h->leaf_mode == BVH_LEAF_COMPACT) {
        k_leaf_compact<<<grid_for(ls.n), kBlock, 0, s>>>(ls.verts, ls.n_verts, ls.tris, ls.perm,
                                                          ls.n, static_cast<bvh_tri *>(h->leaf));
    } else {
        BVH_HIP_TRY(hipMemcpyAsync(h->leaf, ls.perm, (size_t)ls.n * sizeof(int32_t),
                                   hipMemcpyDeviceToDevice, s));
        BVH_HIP_TRY(hipMemcpyAsync(h->verts, ls.verts, (size_t)ls.n_verts * 3 * sizeof(float),
                                   hipMemcpyDeviceToDevice, s));
        BVH_HIP_TRY(hipMemcpyAsync(h->tris, ls.tris, (size_t)ls.n * 3 * sizeof(int32_t),
                                   hipMemcpyDeviceToDevice, s));
    }
    return check_launch("leaf packing");
}

// Wide node counts of earlier builds, keyed by device, layout, leaf size,
// builder and triangle count.  A build whose key was seen allocates its node
// block up front (count + 1/64 + 64 nodes) while queued kernels run, and
// packs straight into it; without a hint, or when the tree turns out larger,
// the nodes go to the work area and into an exact block after the last level
// (a host-blocking hipMalloc with the GPU idle, then a copy).  Repeated
// builds of one mesh, as in per-frame rebuilds, hit the hint.
class NodeCountHints {
  public:
    using Key = std::array<int64_t, 5>;
    int64_t get(const Key &k) {
        std::lock_guard<std::mutex> g(mu_);
        auto it = map_.find(k);
        return it == map_.end() ? 0 : it->second;
    }
    void put(const Key &k, int64_t v) {
        std::lock_guard<std::mutex> g(mu_);
        if (map_.size() >= kMaxEntries) map_.clear();
        map_[k] = v;
    }

  private:
    static constexpr size_t kMaxEntries = 4096;
    std::mutex mu_;
    std::map<Key, int64_t> map_;
};

NodeCountHints &node_count_hints() {
    static NodeCountHints hints;
    return hints;
}

NodeCountHints::Key node_hint_key(const bvh_handle_s *h) {
    return NodeCountHints::Key{h->device, h->layout, h->leaf_size, h->builder, h->n_tris};
}

// The node block of a wide layout, sized from the hint (none without one);
// called while queued kernels keep the GPU busy.
int32_t alloc_node_block_ahead(bvh_handle_s *h) {
    const int64_t hint = node_count_hints().get(node_hint_key(h));
    if (hint <= 0) return BVH_OK;
    const int64_t want = std::min<int64_t>(std::max<int64_t>(1, h->n_tris - 1), hint + hint / 64 + 64);
    if (block_alloc(h->device, (size_t)want * h->node_bytes, &h->node_block) != hipSuccess) {
        (void)hipGetLastError();  // no block ahead: the exact one comes after packing
        return BVH_OK;
    }
    h->node_block_cap = (uint32_t)want;
    return BVH_OK;
}

// A second stream per host thread and device (default priority), with two
// events, for build work off the critical path: the leaf data needs only the
// sorted order, so it runs beside the hierarchy and packing kernels, which
// leave much of the GPU idle.  Null stream when creation fails.
struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t ready = nullptr, done = nullptr;
};

SideStream *side_stream(int device) {
    static thread_local std::map<int, SideStream> streams;
    SideStream &ss = streams[device];
    if (!ss.stream) {
        if (hipStreamCreateWithFlags(&ss.stream, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&ss.ready, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&ss.done, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            ss = SideStream{};
            return nullptr;
        }
    }
    return &ss;
}

// The wide packing does not wait for the whole build so far: the leaf data
// and the child lists (which need no count) are queued first, then the host
// reads the leaf count from the word the collapse scan writes (*nleaf_word,
// host-mapped) while those kernels run.  cand_all / ni_all hold max(n-1, 1)
// lists of K.  The plan, placement and writing kernels are queued at once;
// the host waits only for the final node count.
template <int Layout>
int32_t pack_wide(TreeView tv, volatile uint32_t *nleaf_word, int32_t *cand_all, uint32_t *ni_all,
                  BuildInfo *info, bvh_handle_s *h, const LeafSource &ls, hipStream_t s) {
    constexpr int K = WideOut<Layout>::K;
    const uint32_t m = std::max<uint32_t>(1, (uint32_t)tv.n - 1);  // binary nodes with a list
    (void)ls;  // the leaf data is already queued (build_impl, on the side stream)
    k_wide_open_all<K><<<grid_for(m), kBlock, 0, s>>>(tv, m, cand_all, ni_all);
    BVH_TRY(check_launch("wide packing (child lists)"));
    uint32_t n_leaves = 0;
    BVH_TRY(wait_host_word(nleaf_word, s, &n_leaves));
    if (n_leaves < 1 || n_leaves > (uint32_t)tv.n)
        return set_error(BVH_EHIP, "bvh_build: internal error (leaf count %u)", n_leaves);
    h->n_leaves = n_leaves;
    const uint32_t cap = std::max<uint32_t>(1, n_leaves - 1);  // alive interior nodes (or 1)
    constexpr uint32_t kRoots = K * kTopMaxFrontier;
    const size_t nq = std::max<size_t>(1, (size_t)tv.n);
    uint8_t *wnodes;
    WidePlan p;
    Arena arena;
    arena.request(&wnodes, (size_t)cap * h->node_bytes);
    arena.request(&p.t_node, kTopMaxNodes);
    arena.request(&p.t_aux, kTopMaxNodes);
    arena.request(&p.t_noff, kTopMaxNodes);
    arena.request(&p.f_node, kRoots);
    arena.request(&p.f_aux, kRoots);
    arena.request(&p.f_size, kRoots);
    arena.request(&p.f_off, kRoots);
    arena.request(&p.f_q0, kRoots);
    arena.request(&p.s_node, nq);
    arena.request(&p.s_aux, nq);
    arena.request(&p.s_noff, nq);
    arena.request(&p.meta, 4);
    BVH_TRY(arena.bind(s, kAreaBuildWide));
    uint32_t *hw = host_words();
    if (!hw) return set_error(BVH_ENOMEM, "hipHostMalloc failed");
    volatile uint32_t *vw = hw;
    vw[0] = kPending;
    NodeSink sink{static_cast<uint8_t *>(h->node_block.ptr), h->node_block.ptr ? h->node_block_cap : 0u,
                  wnodes, (uint32_t)h->node_bytes};
    const NodeCountHints::Key key = node_hint_key(h);
    const bool whole = cap <= kTopMaxFrontier;
    k_wide_plan_top<K><<<1, kTopThreads, 0, s>>>(cand_all, ni_all, p, whole, cap, info, hw);
    if (!whole) {
        k_wide_plan_sub<K><<<std::min(kRoots, kPlanBlocks), kSubThreads, 0, s>>>(tv, cand_all, ni_all,
                                                                               p, info);
        k_wide_place<<<1, kPlaceThreads, 0, s>>>(p, cap, info, hw);
    }
    k_wide_write<Layout><<<grid_for((uint64_t)cap * K), kBlock, 0, s>>>(tv, cand_all, p, cap, sink, info);
    // the stack and depth bounds, queued before the host waits for the count
    k_fold_max_slots<<<1, kBlock, 0, s>>>(tv.stack_slots, tv.depth_slots, info);
    BVH_TRY(check_launch("wide packing"));
    uint32_t base = 0;
    BVH_TRY(wait_host_word(vw, s, &base));
    if (base > cap) return set_error(BVH_EHIP, "wide packing overflow");
    h->n_nodes = base;
    // the wide traversal kernels address node fields with 32-bit byte offsets
    if ((uint64_t)base * (uint64_t)h->node_bytes >= (1ull << 32))
        return set_error(BVH_EUNSUPPORTED,
                         "bvh_build: wide node buffer of %llu bytes exceeds 4 GiB (raise leaf_size)",
                         (unsigned long long)base * (unsigned long long)h->node_bytes);
    node_count_hints().put(key, base);
    if (sink.spec && base <= sink.spec_cap) {  // every node is in place
        h->nodes = h->node_block.ptr;
        return BVH_OK;
    }
    DeviceBlock spec = h->node_block;  // too small (or absent): move into an exact block
    h->node_block = DeviceBlock{};
    const int32_t rc = alloc_node_block(h, base);
    if (rc == BVH_OK) {
        const size_t nb0 = (size_t)std::min(base, sink.spec_cap) * h->node_bytes;
        const size_t all = (size_t)base * h->node_bytes;
        hipError_t e = hipSuccess;
        if (nb0 > 0) e = hipMemcpyAsync(h->nodes, spec.ptr, nb0, hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(static_cast<uint8_t *>(h->nodes) + nb0, wnodes + nb0, all - nb0,
                               hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess && spec.ptr) e = hipStreamSynchronize(s);
        if (spec.ptr) (void)hipFree(spec.ptr);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return set_error(BVH_EHIP, "wide packing: node copy failed: %s", hipGetErrorString(e));
        }
        return BVH_OK;
    }
    if (spec.ptr) (void)hipFree(spec.ptr);
    return rc;
}

// ---------------------------------------------------------------------------
// a4 alternative: binned-SAH topology (32 bins per axis; Sec. 9.2.1).  Top
// down: a node bins its primitives' centroids along each axis over their
// exact bounds, takes the cheapest split A(L) N(L) + A(R) N(R) (A = half
// the surface area of a side's union box; ties to the lower axis, then the
// lower split), and partitions stably; coincident centroids split at the
// index median.  Splitting goes down to single primitives, and the result
// is the same tree view the Karras hierarchy produces (internal nodes
// 0 .. n-2, primitive at leaf position k is node n-1+k, ranges of the
// permutation), so boxes, collapse and packing follow unchanged.
//
// Internal node ids: a node whose split falls between leaf positions m-1
// and m gets id m-1 (unique), except that the root takes id 0 and the node
// with natural id 0 takes the root's natural id.
//
// Large nodes (more than kSahSmall primitives) are processed level by level,
// in chunks of kSahChunk primitives with a block each: binning, one wave per
// node for the sweep, then a stable partition, which also takes the centroid
// bounds of the children that the next level bins.  A chunk's bins hold what
// the partition needs of the other chunks (how many of their primitives go
// left), so no flag is written and nothing is scanned over the whole array.
// Nodes of at most kSahMid primitives leave the levels: a workgroup each takes
// them down to small ones.
// A level costs its launches' latency rather than memory traffic: 300,000
// triangles spend 430 us on 13 levels (with separate launches for bounds, flags,
// their scan and the counts' publication, 58 us a level).  Nodes of at most
// kSahSmall primitives are finished by one wave each with the primitives held
// in the lanes.
// ---------------------------------------------------------------------------
constexpr int kSahBins = 32;
constexpr uint32_t kSahSmall = 64;
constexpr uint32_t kSahMid = 1024;
constexpr uint32_t kSahChunk = 2048;
constexpr int kSahMaxLevels = kStackMax + 1;
constexpr uint32_t kSahBinWords = 3 * kSahBins * 7;  // per node: count + ordered box per bin

struct SahTask {
    uint32_t first, count;
    int32_t parent;  // id of the parent (-1: root)
    uint32_t side;   // 0: left child of the parent, 1: right
};

struct SahSplit {
    int32_t axis;  // split axis (0 for an index-median split)
    int32_t k;     // last bin of the left side (-1: index median)
    uint32_t nl;   // primitives on the left
    uint32_t id;   // the node's id
    uint32_t slot[2];  // per side: the child's task in the next level (kNoSlot: none)
};
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;

// Floats as order-preserving ints, so min/max can use integer atomics.
__device__ inline int f2o(float f) {
    const int i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7FFFFFFF;
}
__device__ inline float o2f(int i) { return __int_as_float(i >= 0 ? i : i ^ 0x7FFFFFFF); }

__device__ inline float sah_centroid(const Box &b, int a) {
    const float lo = a == 0 ? b.lo.x : (a == 1 ? b.lo.y : b.lo.z);
    const float hi = a == 0 ? b.hi.x : (a == 1 ? b.hi.y : b.hi.z);
    return 0.5f * lo + 0.5f * hi;
}

// Binning frame of one axis: valid when the centroid extent is positive and
// finite; then bin(c) = min(31, trunc((c - lo) * scale)), scale = 32 / ext.
struct SahFrame {
    float4 lo, scale;  // per axis in x, y, z
    uint32_t valid;    // bit a: axis a can be binned
    // the axis is picked among register values, never by indexing memory, so
    // a run-time axis does not send the frame to scratch memory
    __device__ bool ok(int a) const { return (valid >> a) & 1u; }
};

__device__ inline float axis_of(const float4 v, int a) { return a == 0 ? v.x : (a == 1 ? v.y : v.z); }

__device__ inline SahFrame sah_frame(const float *cl, const float *ch) {
    SahFrame f;
    float lo[3], sc[3];
    f.valid = 0;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const float ext = ch[a] - cl[a];
        const bool v = ext > 0.0f && !isinf(ext);
        f.valid |= (v ? 1u : 0u) << a;
        lo[a] = cl[a];
        sc[a] = v ? __fdiv_rn((float)kSahBins, ext) : 0.0f;
    }
    f.lo = make_float4(lo[0], lo[1], lo[2], 0.0f);
    f.scale = make_float4(sc[0], sc[1], sc[2], 0.0f);
    return f;
}

__device__ inline int sah_bin(const SahFrame f, int a, float c) {
    const float4 lo4 = f.lo, sc4 = f.scale;
    const int b = (int)((c - axis_of(lo4, a)) * axis_of(sc4, a));  // c >= lo: b >= 0 for finite input
    return b < 0 ? 0 : (b < kSahBins - 1 ? b : kSahBins - 1);
}

__device__ inline float half_area3(float lx, float ly, float lz, float hx, float hy, float hz) {
    const float dx = hx - lx, dy = hy - ly, dz = hz - lz;
    return (dx * dy + dy * dz) + dz * dx;
}

// Cheapest splits of two axes from their 32 bins each: bin k of one axis in
// lane k, of the other in lane 32 + k (the scans stay within each half): count
// and box as floats; empty bins hold an empty box.  Per half, in every lane:
// the lowest cost (+inf when no split leaves both sides non-empty), the lowest
// bin among equal costs (-1 when no split has a finite cost) and its left count.
__device__ inline void sah_sweep2(uint32_t cnt, float lx, float ly, float lz, float hx, float hy,
                                  float hz, float &cost0, int &k0, uint32_t &nl0, float &cost1,
                                  int &k1, uint32_t &nl1) {
    const int lane = threadIdx.x & (kWave - 1);
    const int hl = lane & (kSahBins - 1);  // the bin in the lane's half
    const auto add = [](uint32_t x, uint32_t y) { return x + y; };
    const auto mn = [](float x, float y) { return fminf(x, y); };
    const auto mx = [](float x, float y) { return fmaxf(x, y); };
    const uint32_t pc = half_scan<uint32_t>(cnt, 0u, add);
    const uint32_t sc = half_suffix_scan<uint32_t>(cnt, 0u, add, lane);
    const float in[6] = {lx, ly, lz, hx, hy, hz};
    float p[6], q[6];
#pragma unroll
    for (int j = 0; j < 3; j++) {
        p[j] = half_scan<float>(in[j], INFINITY, mn);
        q[j] = half_suffix_scan<float>(in[j], INFINITY, mn, lane);
        p[3 + j] = half_scan<float>(in[3 + j], -INFINITY, mx);
        q[3 + j] = half_suffix_scan<float>(in[3 + j], -INFINITY, mx, lane);
    }
    // the right side of split k is the suffix from bin k + 1 (wave_shl:1;
    // the last bin of each half has no split)
    const uint32_t rc = dpp<0x130, 0xf>(0u, sc);
    float r[6];
#pragma unroll
    for (int j = 0; j < 6; j++) r[j] = dpp<0x130, 0xf>(j < 3 ? INFINITY : -INFINITY, q[j]);
    float cost = INFINITY;
    if (hl < kSahBins - 1 && pc > 0 && rc > 0)
        cost = half_area3(p[0], p[1], p[2], p[3], p[4], p[5]) * (float)pc +
               half_area3(r[0], r[1], r[2], r[3], r[4], r[5]) * (float)rc;
    const float m = half_scan<float>(cost, INFINITY, mn);  // each half's minimum at its last lane
    cost0 = readlane_t(m, kSahBins - 1);
    cost1 = readlane_t(m, kWave - 1);
    const uint64_t at = __builtin_amdgcn_ballot_w64(hl < kSahBins - 1 && cost == (lane < kSahBins ? cost0 : cost1));
    const uint32_t at0 = (uint32_t)at, at1 = (uint32_t)(at >> 32);
    k0 = (cost0 < INFINITY && at0 != 0) ? (int)__builtin_ctz(at0) : -1;
    k1 = (cost1 < INFINITY && at1 != 0) ? (int)__builtin_ctz(at1) : -1;
    nl0 = readlane_t(pc, k0 < 0 ? 0 : k0);
    nl1 = readlane_t(pc, kSahBins + (k1 < 0 ? 0 : k1));
}

// Id of the node that splits at leaf position m (m-1 naturally; see above).
__device__ inline uint32_t sah_node_id(uint32_t m, bool is_root, uint32_t root_nat) {
    if (is_root) return 0u;
    const uint32_t nat = m - 1u;
    return nat == 0u ? root_nat : nat;
}

struct SahTree {
    int32_t *ileft, *iright, *parent;
    uint32_t *ifirst, *icount;
    uint8_t *iaxis;
    int n;
};

// Records node id (range, axis, parent link) and links its leaf children.
__device__ inline void sah_write_node(const SahTree &tr, uint32_t id, uint32_t first,
                                      uint32_t count, int axis, uint32_t nl, int32_t parent,
                                      uint32_t side) {
    tr.ifirst[id] = first;
    tr.icount[id] = count;
    tr.iaxis[id] = (uint8_t)axis;
    tr.parent[id] = parent;
    if (parent >= 0) (side ? tr.iright : tr.ileft)[parent] = (int32_t)id;
    if (nl == 1) {
        const int32_t leaf = tr.n - 1 + (int32_t)first;
        tr.ileft[id] = leaf;
        tr.parent[leaf] = (int32_t)id;
    }
    if (count - nl == 1) {
        const int32_t leaf = tr.n - 1 + (int32_t)(first + nl);
        tr.iright[id] = leaf;
        tr.parent[leaf] = (int32_t)id;
    }
}

// Per-level state of the large-node phase (device).
struct SahLevel {
    const SahTask *task;      // this level's nodes
    const uint32_t *chunk;    // per chunk: task index
    const uint32_t *cstart;   // per chunk: first position
    int *cb;                  // per task: centroid bounds (ordered ints, lo xyz, hi xyz)
    int *bins;                // per task: kSahBinWords
    SahSplit *split;          // per task
    uint32_t ntask;
    const uint32_t *tc0;      // per task: its first chunk (a task's chunks are consecutive)
    int *cbins;               // per chunk: kSahBinWords (the chunk's partial bins)
    int *gbins;               // merge groups > 1: per task and group, kSahBinWords
    uint32_t groups;          // chunk groups per task in the merge (1 or kMergeGroups)
    uint32_t *ccnt;           // per chunk: kSahCounts running counts over each axis's bins
    uint32_t *cleft;          // per chunk of a task with several: left primitives before it
};
constexpr uint32_t kSahCounts = 3 * kSahBins;
constexpr int kSahRows = kSahChunk / kBlock;  // primitives per thread of a chunk's block
static_assert(kSahRows * kBlock == (int)kSahChunk, "a chunk is a whole number of rows");

// Chunk groups of a task of nch chunks in a level merged with `groups` groups.
__device__ inline uint32_t merge_groups(uint32_t nch, uint32_t groups) { return min(nch, groups); }

// Centroid bounds of a block's primitives into a task's words: v of each
// thread (lo xyz, hi xyz), red scratch of the block.  Every thread calls it.
__device__ inline void sah_fold_bounds(const float (&v)[6], float (*red)[kBlock / kWave], int *cb) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    __syncthreads();  // red may hold an earlier fold's values
#pragma unroll
    for (int j = 0; j < 6; j++) {
        const float r = j < 3 ? wave_min(v[j]) : wave_max(v[j]);
        if (lane == 0) red[j][w] = r;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int j = threadIdx.x;
        float r = red[j][0];
        for (int k = 1; k < kBlock / kWave; k++) r = j < 3 ? fminf(r, red[j][k]) : fmaxf(r, red[j][k]);
        if (j < 3) atomicMin(&cb[j], f2o(r));
        else atomicMax(&cb[j], f2o(r));
    }
}

__device__ inline void sah_clear_bounds(int *cb) {
#pragma unroll
    for (int j = 0; j < 6; j++) cb[j] = f2o(j < 3 ? INFINITY : -INFINITY);
}

// The root's centroid bounds (k_sah_init has cleared them).
__global__ __launch_bounds__(kBlock) void k_sah_bounds(uint32_t n, const Box *pbox, int *cb) {
    __shared__ float red[6][kBlock / kWave];
    const uint32_t p0 = blockIdx.x * kSahChunk, p1 = min(p0 + kSahChunk, n);
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (uint32_t p = p0 + threadIdx.x; p < p1; p += kBlock) {
        const Box b = pbox[p];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const float c = sah_centroid(b, a);
            v[a] = fminf(v[a], c);
            v[3 + a] = fmaxf(v[3 + a], c);
        }
    }
    sah_fold_bounds(v, red, cb);
}

__device__ inline SahFrame sah_task_frame(const int *cb) {
    float cl[3], ch[3];
    for (int a = 0; a < 3; a++) {
        cl[a] = o2f(cb[a]);
        ch[a] = o2f(cb[3 + a]);
    }
    return sah_frame(cl, ch);
}

// Binning of one chunk.  Neighbouring primitives (in the current order)
// mostly fall in one bin, so the lanes of a wave instruction would update the
// same LDS words: the block keeps kBinCopies copies of the bins, lane i using
// copy i % kBinCopies (copies a bank apart), which divides those conflicts by
// kBinCopies; the copies are combined when the chunk is done.
constexpr int kBinCopies = 8;
constexpr int kBinCopyStride = kSahBinWords + 1;  // odd: copies in different banks

__global__ __launch_bounds__(kBlock) void k_sah_bin(SahLevel lv, const uint32_t *ord,
                                                    const Box *pbox) {
    __shared__ int sb[kBinCopies * kBinCopyStride];
    const uint32_t t = lv.chunk[blockIdx.x];
    const SahTask tk = lv.task[t];
    const uint32_t p0 = lv.cstart[blockIdx.x], p1 = min(p0 + kSahChunk, tk.first + tk.count);
    // every box is asked for before the bins are cleared
    uint32_t prim[kSahRows];
    Box box[kSahRows];
#pragma unroll
    for (int r = 0; r < kSahRows; r++) {
        const uint32_t p = p0 + r * kBlock + threadIdx.x;
        if (p < p1) prim[r] = ord[p];
    }
#pragma unroll
    for (int r = 0; r < kSahRows; r++)
        if (p0 + r * kBlock + threadIdx.x < p1) box[r] = pbox[prim[r]];
    const SahFrame f = sah_task_frame(lv.cb + 6 * t);
    const int inf = f2o(INFINITY), ninf = f2o(-INFINITY);
    for (uint32_t i = threadIdx.x; i < kBinCopies * kBinCopyStride; i += kBlock) {
        const uint32_t w = (i % kBinCopyStride) % 7;
        sb[i] = w == 0 ? 0 : (w <= 3 ? inf : ninf);
    }
    __syncthreads();
    int *mine = sb + (threadIdx.x % kBinCopies) * kBinCopyStride;
#pragma unroll
    for (int r = 0; r < kSahRows; r++) {
        if (p0 + r * kBlock + threadIdx.x >= p1) break;
        const Box b = box[r];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            if (!f.ok(a)) continue;
            int *bin = mine + (a * kSahBins + sah_bin(f, a, sah_centroid(b, a))) * 7;
            atomicAdd(bin, 1);
            atomicMin(bin + 1, f2o(b.lo.x));
            atomicMin(bin + 2, f2o(b.lo.y));
            atomicMin(bin + 3, f2o(b.lo.z));
            atomicMax(bin + 4, f2o(b.hi.x));
            atomicMax(bin + 5, f2o(b.hi.y));
            atomicMax(bin + 6, f2o(b.hi.z));
        }
    }
    __syncthreads();
    // the chunk's partial bins, every word (k_sah_merge combines a task's
    // chunks; device atomics from every chunk of a large task into one set of
    // words serialised across the XCDs)
    int *cbin = lv.cbins + (size_t)blockIdx.x * kSahBinWords;
    for (uint32_t i = threadIdx.x; i < kSahBinWords; i += kBlock) {
        const uint32_t kind = i % 7;
        int v = sb[i];
        for (int c = 1; c < kBinCopies; c++) {
            const int x = sb[c * kBinCopyStride + i];
            v = kind == 0 ? v + x : (kind <= 3 ? min(v, x) : max(v, x));
        }
        cbin[i] = v;
        if (kind == 0) sb[i] = v;  // word i of the copies is this thread's
    }
    __syncthreads();
    if (threadIdx.x < 2 * kWave) {  // whole waves; a half of a wave per axis
        const uint32_t c = threadIdx.x < kSahCounts ? (uint32_t)sb[threadIdx.x * 7] : 0u;
        const uint32_t run = half_scan<uint32_t>(c, 0u, [](uint32_t x, uint32_t y) { return x + y; });
        if (threadIdx.x < kSahCounts) lv.ccnt[(size_t)blockIdx.x * kSahCounts + threadIdx.x] = run;
    }
}

// bins of task t = the combination of its chunks' partial bins: counts
// added, ordered-int lower corners by minimum, upper corners by maximum (the
// same integers in any order).  Block (t, g) combines chunk group g of task
// t: with one group it writes the task's bins, with several its group's
// partial bins (sah_split_node combines the groups; levels of few, large
// tasks use several, so that one block does not read all the chunks of the
// root).  A task of one chunk is read from its chunk directly.
constexpr uint32_t kMergeGroups = 16;
constexpr uint32_t kMergeGroupTasks = 256;  // most tasks of a level merged with several groups

__device__ inline int bin_combine(uint32_t kind, int v, int x) {
    return kind == 0 ? v + x : (kind <= 3 ? min(v, x) : max(v, x));
}

__global__ __launch_bounds__(kBlock) void k_sah_merge(SahLevel lv) {
    const uint32_t t = blockIdx.x, g = blockIdx.y;
    const uint32_t nch = (lv.task[t].count + kSahChunk - 1) / kSahChunk, c0 = lv.tc0[t];
    const uint32_t ng = merge_groups(nch, lv.groups);
    if (nch < 2 || g >= ng) return;
    const uint32_t j0 = (uint32_t)((uint64_t)g * nch / ng), j1 = (uint32_t)((uint64_t)(g + 1) * nch / ng);
    int *dst = ng > 1 ? lv.gbins + ((size_t)t * kMergeGroups + g) * kSahBinWords
                      : lv.bins + (size_t)t * kSahBinWords;
    for (uint32_t w = threadIdx.x; w < (uint32_t)kSahBinWords; w += kBlock) {
        const int *src = lv.cbins + (size_t)c0 * kSahBinWords + w;
        const uint32_t kind = w % 7;  // 0: count, 1-3: lower corner, 4-6: upper corner
        int v = src[(size_t)j0 * kSahBinWords];
        uint32_t j = j0 + 1;
        for (; j + 4 <= j1; j += 4) {  // four independent loads in flight
            const int x0 = src[(size_t)j * kSahBinWords], x1 = src[(size_t)(j + 1) * kSahBinWords];
            const int x2 = src[(size_t)(j + 2) * kSahBinWords], x3 = src[(size_t)(j + 3) * kSahBinWords];
            v = bin_combine(kind, v, bin_combine(kind, bin_combine(kind, x0, x1), bin_combine(kind, x2, x3)));
        }
        for (; j < j1; j++) v = bin_combine(kind, v, src[(size_t)j * kSahBinWords]);
        dst[w] = v;
    }
}

// The cheapest split of a node of `count` primitives from its bins: lane l has
// bin l % 32 of x (lanes 0-31) or y in w0, of z in w1 (7 words each).  Without
// a split of finite cost, the index median: axis 0, bk -1.
__device__ inline void sah_choose(const SahFrame f, const int (&w0)[7], const int (&w1)[7],
                                  uint32_t count, int &axis, int &bk, uint32_t &nl) {
    const bool v0 = f.ok(0), v1 = f.ok(1), v2 = f.ok(2);
    float best = INFINITY;
    axis = bk = -1;
    nl = 0;
    // the costs are compared in axis order with a strict <: a lower axis wins a tie
    if (v0 || v1) {
        float cx, cy;
        int kx, ky;
        uint32_t lx, ly;
        sah_sweep2((uint32_t)w0[0], o2f(w0[1]), o2f(w0[2]), o2f(w0[3]), o2f(w0[4]), o2f(w0[5]),
                   o2f(w0[6]), cx, kx, lx, cy, ky, ly);
        if (v0 && cx < best) {
            best = cx;
            axis = 0;
            bk = kx;
            nl = lx;
        }
        if (v1 && cy < best) {
            best = cy;
            axis = 1;
            bk = ky;
            nl = ly;
        }
    }
    if (v2) {
        float cz, unused_c;
        int kz, unused_k;
        uint32_t lz, unused_l;
        sah_sweep2((uint32_t)w1[0], o2f(w1[1]), o2f(w1[2]), o2f(w1[3]), o2f(w1[4]), o2f(w1[5]),
                   o2f(w1[6]), cz, kz, lz, unused_c, unused_k, unused_l);
        if (cz < best) {
            axis = 2;
            bk = kz;
            nl = lz;
        }
    }
    if (axis < 0) {
        axis = 0;
        bk = -1;
        nl = count / 2;
    }
}

// The sweep and record of node t (one wave); leaves its task, id and split
// (but for the slots) in tk and sp, the same in every lane.
__device__ inline void sah_split_node(SahLevel lv, SahTree tr, uint32_t *root_nat, bool root_level,
                                      uint32_t t, int lane, SahTask &tk, SahSplit &sp) {
    tk = lv.task[t];
    const uint32_t nch = (tk.count + kSahChunk - 1) / kSahChunk, c0 = lv.tc0[t];
    const uint32_t ng = nch < 2 ? 1u : merge_groups(nch, lv.groups);
    // one chunk: its chunk's bins; several in one group: the merged bins;
    // several groups: the groups' partial bins, combined here
    const int *gb = nch < 2 ? lv.cbins + (size_t)c0 * kSahBinWords
                            : (ng > 1 ? lv.gbins + (size_t)t * kMergeGroups * kSahBinWords
                                      : lv.bins + (size_t)t * kSahBinWords);
    const SahFrame f = sah_task_frame(lv.cb + 6 * t);
    // x's bins in lanes 0-31 and y's in lanes 32-63, then z's in lanes 0-31
    const int *bin0 = gb + lane * 7, *bin1 = gb + (2 * kSahBins + (lane & (kSahBins - 1))) * 7;
    int w0[7], w1[7];
#pragma unroll
    for (int j = 0; j < 7; j++) {
        w0[j] = bin0[j];
        w1[j] = bin1[j];
    }
#pragma unroll 4
    for (uint32_t g = 1; g < ng; g++) {
        const size_t at = (size_t)g * kSahBinWords;
#pragma unroll
        for (int j = 0; j < 7; j++) {
            w0[j] = bin_combine((uint32_t)j, w0[j], bin0[at + j]);
            w1[j] = bin_combine((uint32_t)j, w1[j], bin1[at + j]);
        }
    }
    int axis, bk;
    uint32_t nl;
    sah_choose(f, w0, w1, tk.count, axis, bk, nl);
    const uint32_t m = tk.first + nl;
    if (root_level && lane == 0) *root_nat = m - 1;
    const uint32_t rn = root_level ? m - 1 : *root_nat;
    sp = SahSplit{axis, bk, nl, sah_node_id(m, tk.parent < 0, rn), {kNoSlot, kNoSlot}};
    if (nch > 1 && bk >= 0) {  // the left primitives before each chunk
        uint32_t carry = 0;
        for (uint32_t j0 = 0; j0 < nch; j0 += kWave) {
            const uint32_t j = j0 + lane;
            const uint32_t v = j < nch ? lv.ccnt[(size_t)(c0 + j) * kSahCounts + axis * kSahBins + bk] : 0u;
            uint32_t run = half_scan<uint32_t>(v, 0u, [](uint32_t x, uint32_t y) { return x + y; });
            if (lane >= kSahBins) run += readlane_t(run, kSahBins - 1);
            if (j < nch) lv.cleft[c0 + j] = carry + run - v;
            carry += readlane_t(run, kWave - 1);
        }
    }
    if (lane == 0) sah_write_node(tr, sp.id, tk.first, tk.count, axis, nl, tk.parent, tk.side);
}

// One wave per node: the sweep over the three axes, then the node's id and
// record, and its children: single primitives are linked here, small ones
// queued for the per-wave finisher, large ones queued (with their chunks)
// for the next level.  The queue slots of a block's nodes are taken with one
// device atomic per queue and block (per-node atomics on the three counters
// serialised across the XCDs: 0.2-0.45 ms per level with thousands of nodes).
// Levels of few nodes use small blocks, which start sooner and spread over the
// GPU (SAH builds of 5,000 to 300,000 triangles 4-7 % faster); levels of many
// use large ones, for fewer atomics (2,000,000 triangles 2 % faster).
constexpr int kSplitFewThreads = 256, kSplitManyThreads = 1024;
constexpr uint32_t kSplitFewTasks = 2048;

template <int kSplitThreads>
__global__ __launch_bounds__(kSplitThreads) void k_sah_split(SahLevel lv, SahTree tr,
                                                             uint32_t *root_nat, bool root_level,
                                                             SahTask *next, uint32_t *next_chunk,
                                                             uint32_t *next_cstart,
                                                             uint32_t *next_tc0, int *next_cb,
                                                             uint32_t *counters, SahTask *small,
                                                             uint32_t *small_count, SahTask *mid,
                                                             uint32_t *mid_count) {
    constexpr int kSplitWaves = kSplitThreads / kWave;
    __shared__ uint32_t need[4][kSplitWaves];  // per wave: small, next tasks, next chunks, middle
    __shared__ uint32_t base[4];
    const int wv = threadIdx.x / kWave;
    const uint32_t t = blockIdx.x * kSplitWaves + wv;
    const bool live = t < lv.ntask;
    const int lane = threadIdx.x & (kWave - 1);
    SahTask tk{0, 0, -1, 0};
    SahSplit sp{0, -1, 0, 0, {kNoSlot, kNoSlot}};
    if (live) sah_split_node(lv, tr, root_nat, root_level, t, lane, tk, sp);
    const uint32_t nl = sp.nl;
    // the node's children that need queue slots
    const uint32_t cf[2] = {tk.first, tk.first + nl}, cc[2] = {nl, tk.count - nl};
    uint32_t ns = 0, nn = 0, nc = 0, nm = 0;
    if (live) {
        for (int sd = 0; sd < 2; sd++) {
            if (cc[sd] < 2) continue;
            if (cc[sd] <= kSahSmall) {
                ns++;
            } else if (cc[sd] <= kSahMid) {
                nm++;
            } else {
                nn++;
                nc += (cc[sd] + kSahChunk - 1) / kSahChunk;
            }
        }
    }
    if (lane == 0) {
        need[0][wv] = ns;
        need[1][wv] = nn;
        need[2][wv] = nc;
        need[3][wv] = nm;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        uint32_t tot = 0;
        for (int w = 0; w < kSplitWaves; w++) tot += need[threadIdx.x][w];
        uint32_t *ctr = threadIdx.x == 0 ? small_count
                                         : (threadIdx.x == 3 ? mid_count : &counters[threadIdx.x - 1]);
        base[threadIdx.x] = tot ? atomicAdd(ctr, tot) : 0u;
    }
    __syncthreads();
    if (!live || lane != 0) return;
    uint32_t so = base[0], no = base[1], co = base[2], mo = base[3];
    for (int w = 0; w < wv; w++) {
        so += need[0][w];
        no += need[1][w];
        co += need[2][w];
        mo += need[3][w];
    }
    for (int sd = 0; sd < 2; sd++) {
        if (cc[sd] < 2) continue;
        const SahTask ch{cf[sd], cc[sd], (int32_t)sp.id, (uint32_t)sd};
        if (cc[sd] <= kSahSmall) {
            small[so++] = ch;
        } else if (cc[sd] <= kSahMid) {
            mid[mo++] = ch;
        } else {
            const uint32_t slot = no++;
            sp.slot[sd] = slot;
            next[slot] = ch;
            sah_clear_bounds(next_cb + 6 * (size_t)slot);
            next_tc0[slot] = co;
            const uint32_t nch = (cc[sd] + kSahChunk - 1) / kSahChunk;
            for (uint32_t j = 0; j < nch; j++) {
                next_chunk[co + j] = slot;
                next_cstart[co + j] = cf[sd] + j * kSahChunk;
            }
            co += nch;
        }
    }
    lv.split[t] = sp;
}

// The stable partition of one chunk: each wave takes consecutive rows of it, so
// a primitive's rank among the left ones is that of the chunk (cleft), of the
// waves before and of the lanes and rows before.  Also folds the centroid
// bounds of the children that the next level bins, and the first block tells
// the host the next level's sizes (final since the split), so that the host's
// answer overlaps the partition.
__global__ __launch_bounds__(kBlock) void k_sah_scatter(SahLevel lv, const uint32_t *ord,
                                                        const Box *pbox, uint32_t *ord_next,
                                                        uint32_t *perm, int *next_cb,
                                                        const uint32_t *counters,
                                                        const uint32_t *mid_count, uint32_t *host,
                                                        uint32_t *err) {
    constexpr int W = kBlock / kWave;
    __shared__ float red[6][W];
    __shared__ uint32_t wleft[W];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        host[0] = counters[0];
        host[1] = counters[1];
        host[2] = *mid_count;
        __threadfence_system();  // the host polls the words
    }
    const uint32_t t = lv.chunk[blockIdx.x];
    const SahTask tk = lv.task[t];
    const SahSplit sp = lv.split[t];
    const uint32_t p0 = lv.cstart[blockIdx.x], p1 = min(p0 + kSahChunk, tk.first + tk.count);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t rows = (p1 - p0 + kBlock - 1) / kBlock;
    const uint32_t q0 = p0 + (uint32_t)w * rows * kWave + lane;  // row r: q0 + r * kWave
    uint32_t prim[kSahRows];
    Box box[kSahRows];
#pragma unroll
    for (int r = 0; r < kSahRows; r++) {
        const uint32_t p = q0 + r * kWave;
        if (r < (int)rows && p < p1) prim[r] = ord[p];
    }
#pragma unroll
    for (int r = 0; r < kSahRows; r++)
        if (r < (int)rows && q0 + r * kWave < p1) box[r] = pbox[prim[r]];
    const SahFrame f = sah_task_frame(lv.cb + 6 * t);
    float v[2][6];
#pragma unroll
    for (int j = 0; j < 6; j++) v[0][j] = v[1][j] = j < 3 ? INFINITY : -INFINITY;
    uint64_t lmask[kSahRows];
    uint32_t mine = 0;
#pragma unroll
    for (int r = 0; r < kSahRows; r++) {
        lmask[r] = 0;
        if (r >= (int)rows) break;  // the same in the block
        const uint32_t p = q0 + r * kWave;
        bool left = false;
        if (p < p1) {
            const float c[3] = {sah_centroid(box[r], 0), sah_centroid(box[r], 1), sah_centroid(box[r], 2)};
            left = sp.k < 0 ? p - tk.first < sp.nl
                            : sah_bin(f, sp.axis, sp.axis == 0 ? c[0] : (sp.axis == 1 ? c[1] : c[2])) <= sp.k;
#pragma unroll
            for (int a = 0; a < 3; a++) {
                v[0][a] = fminf(v[0][a], left ? c[a] : INFINITY);
                v[0][3 + a] = fmaxf(v[0][3 + a], left ? c[a] : -INFINITY);
                v[1][a] = fminf(v[1][a], left ? INFINITY : c[a]);
                v[1][3 + a] = fmaxf(v[1][3 + a], left ? -INFINITY : c[a]);
            }
        }
        lmask[r] = __builtin_amdgcn_ballot_w64(left);
        mine += (uint32_t)__builtin_popcountll(lmask[r]);
    }
    if (lane == 0) wleft[w] = mine;
    __syncthreads();
    // left primitives of the node before this wave's first row
    uint32_t lrank0 = sp.k < 0 ? min(p0 - tk.first, sp.nl)
                               : (tk.count > kSahChunk ? lv.cleft[blockIdx.x] : 0u);
    for (int k = 0; k < w; k++) lrank0 += wleft[k];
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < kSahRows; r++) {
        if (r >= (int)rows) break;
        const uint32_t p = q0 + r * kWave;
        const uint32_t lrank = lrank0 + (uint32_t)__builtin_popcountll(lmask[r] & below);
        lrank0 += (uint32_t)__builtin_popcountll(lmask[r]);
        if (p >= p1) continue;
        const bool left = (lmask[r] >> lane) & 1u;
        const uint32_t dst = left ? tk.first + lrank : tk.first + sp.nl + (p - tk.first - lrank);
        if (dst >= tk.first + tk.count || (left ? lrank >= sp.nl : false)) {
            atomicOr(err, 1u);  // the primitives disagree with the split's count
            continue;
        }
        ord_next[dst] = prim[r];
        const uint32_t child = left ? sp.nl : tk.count - sp.nl;
        if (child <= kSahMid) perm[dst] = prim[r];
    }
    // the same in the block
    if (sp.slot[0] != kNoSlot) sah_fold_bounds(v[0], red, next_cb + 6 * (size_t)sp.slot[0]);
    if (sp.slot[1] != kNoSlot) sah_fold_bounds(v[1], red, next_cb + 6 * (size_t)sp.slot[1]);
}

// Splits tasks of kSahSmall to kSahMid primitives down to small ones: one
// workgroup per task, with its boxes and order in LDS, a wave per node, level
// by level.  The levels of many such nodes cost four launches and a round
// trip to the host each, some 30 us, of which little is work.  Builds of 1,000,
// 5,000, 200,000, 300,000 and 2,000,000 triangles: 376, 532, 768, 1,037, 3,117 ->
// 286, 475, 686, 997, 2,992 us (512 and 1,024 primitives measured the same).
constexpr int kMidThreads = 512;
constexpr int kMidWaves = kMidThreads / kWave;
constexpr uint32_t kMidNodes = kSahMid / (kSahSmall + 1) + 1;  // nodes of a level at most

__global__ __launch_bounds__(kMidThreads) void k_sah_mid(const SahTask *mid, const Box *pbox,
                                                         uint32_t *perm, SahTree tr,
                                                         uint32_t *root_nat_p, SahTask *small,
                                                         uint32_t *small_count, uint32_t *err) {
    __shared__ float s_box[6][kSahMid];
    __shared__ uint32_t s_prim[kSahMid];
    __shared__ uint16_t s_ord[2][kSahMid];  // by level parity: positions in the arrays above
    __shared__ int s_bin[kMidWaves][kSahBinWords];
    __shared__ SahTask s_node[2][kMidNodes];  // ranges within the task
    __shared__ SahTask s_small[kSahMid / 2];
    __shared__ uint32_t s_n[2], s_nsmall, s_root, s_base;
    const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const SahTask tk = mid[blockIdx.x];
    for (uint32_t i = threadIdx.x; i < tk.count; i += kMidThreads) {
        const uint32_t prim = perm[tk.first + i];
        const Box b = pbox[prim];
        s_prim[i] = prim;
        s_ord[0][i] = (uint16_t)i;
        s_box[0][i] = b.lo.x;
        s_box[1][i] = b.lo.y;
        s_box[2][i] = b.lo.z;
        s_box[3][i] = b.hi.x;
        s_box[4][i] = b.hi.y;
        s_box[5][i] = b.hi.z;
    }
    if (threadIdx.x == 0) {
        s_node[0][0] = SahTask{0u, tk.count, tk.parent, tk.side};
        s_n[0] = 1;
        s_n[1] = 0;
        s_nsmall = 0;
        s_root = tk.parent < 0 ? 0u : *root_nat_p;
    }
    __syncthreads();
    int *const bins = s_bin[w];
    for (int cur = 0; s_n[cur] > 0; cur ^= 1) {  // the same in every thread
        for (uint32_t k = w; k < s_n[cur]; k += kMidWaves) {
            const SahTask nd = s_node[cur][k];
            const uint16_t *const ord = s_ord[cur] + nd.first;
            const auto centre = [&](uint32_t p, int a) { return 0.5f * s_box[a][p] + 0.5f * s_box[3 + a][p]; };
            float cl[3], ch[3];
#pragma unroll
            for (int a = 0; a < 3; a++) {
                cl[a] = INFINITY;
                ch[a] = -INFINITY;
            }
            for (uint32_t i = lane; i < nd.count; i += kWave) {
                const uint32_t p = ord[i];
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    const float c = centre(p, a);
                    cl[a] = fminf(cl[a], c);
                    ch[a] = fmaxf(ch[a], c);
                }
            }
#pragma unroll
            for (int a = 0; a < 3; a++) {
                cl[a] = wave_min(cl[a]);
                ch[a] = wave_max(ch[a]);
            }
            const SahFrame f = sah_frame(cl, ch);
            for (uint32_t i = lane; i < kSahBinWords; i += kWave) {
                const uint32_t kind = i % 7;
                bins[i] = kind == 0 ? 0 : f2o(kind <= 3 ? INFINITY : -INFINITY);
            }
            wave_sync();
            for (uint32_t i = lane; i < nd.count; i += kWave) {
                const uint32_t p = ord[i];
                int q[6];
#pragma unroll
                for (int j = 0; j < 6; j++) q[j] = f2o(s_box[j][p]);
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    if (!f.ok(a)) continue;
                    int *bin = bins + (a * kSahBins + sah_bin(f, a, centre(p, a))) * 7;
                    atomicAdd(bin, 1);
#pragma unroll
                    for (int j = 0; j < 3; j++) {
                        atomicMin(bin + 1 + j, q[j]);
                        atomicMax(bin + 4 + j, q[3 + j]);
                    }
                }
            }
            wave_sync();
            int w0[7], w1[7];
#pragma unroll
            for (int j = 0; j < 7; j++) {
                w0[j] = bins[lane * 7 + j];
                w1[j] = bins[(2 * kSahBins + (lane & (kSahBins - 1))) * 7 + j];
            }
            wave_sync();
            int axis, bk;
            uint32_t nl;
            sah_choose(f, w0, w1, nd.count, axis, bk, nl);
            const uint32_t m = tk.first + nd.first + nl;
            const bool is_root = nd.parent < 0;
            const uint32_t id = sah_node_id(m, is_root, is_root ? m - 1 : s_root);
            // stable partition; small children are final in this kernel
            const uint32_t cc[2] = {nl, nd.count - nl};
            uint32_t lrun = 0;
            for (uint32_t i0 = 0; i0 < nd.count; i0 += kWave) {
                const uint32_t i = i0 + lane;
                const bool in = i < nd.count;
                const uint32_t p = in ? ord[i] : 0u;
                const float c = axis == 0 ? centre(p, 0) : (axis == 1 ? centre(p, 1) : centre(p, 2));
                const bool left = in && (bk < 0 ? i < nl : sah_bin(f, axis, c) <= bk);
                const uint64_t lmask = __builtin_amdgcn_ballot_w64(left);
                const uint32_t rank = lrun + (uint32_t)__builtin_popcountll(lmask & below);
                lrun += (uint32_t)__builtin_popcountll(lmask);
                const uint32_t dst = left ? rank : nl + (i - rank);
                if (in && (dst >= nd.count || (left && rank >= nl))) {
                    atomicOr(err, 1u);  // the primitives disagree with the split's count
                } else if (in) {
                    s_ord[cur ^ 1][nd.first + dst] = (uint16_t)p;
                    if ((left ? cc[0] : cc[1]) <= kSahSmall) perm[tk.first + nd.first + dst] = s_prim[p];
                }
            }
            if (lane == 0) {
                if (is_root) {  // the only node of the first level
                    s_root = m - 1;
                    *root_nat_p = m - 1;
                }
                sah_write_node(tr, id, tk.first + nd.first, nd.count, axis, nl, nd.parent, nd.side);
#pragma unroll
                for (int sd = 0; sd < 2; sd++) {
                    const uint32_t cf = sd == 0 ? nd.first : nd.first + nl;
                    if (cc[sd] < 2) continue;
                    if (cc[sd] <= kSahSmall)
                        s_small[atomicAdd(&s_nsmall, 1u)] = SahTask{tk.first + cf, cc[sd], (int32_t)id, (uint32_t)sd};
                    else
                        s_node[cur ^ 1][atomicAdd(&s_n[cur ^ 1], 1u)] = SahTask{cf, cc[sd], (int32_t)id, (uint32_t)sd};
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) s_n[cur] = 0;
        __syncthreads();
    }
    if (threadIdx.x == 0) s_base = s_nsmall ? atomicAdd(small_count, s_nsmall) : 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < s_nsmall; i += kMidThreads) small[s_base + i] = s_small[i];
}

// Finishes tasks of at most kSahSmall primitives, one wave each, with the
// primitives in the lanes (lane i holds position first + i of the task's
// current order).  All nodes of a level are split at once: a lane knows its
// node's lanes [sf, sf + sc), and works out the split whose left side ends
// with its own bin, on each axis, by going through its node's primitives: the
// only splits that the empty bins in between would add are repetitions, and of
// equal splits the lowest bin counts.  A level so takes as many steps as its
// largest node has primitives.  One node after another, each with its 32 bins
// in LDS and their prefix and suffix scans, took 290 us for 300,000 triangles;
// the levels take 200.
__global__ __launch_bounds__(kBlock) void k_sah_small(const SahTask *small, const uint32_t *small_count,
                                                      uint32_t small_cap,
                                                      const Box *pbox, uint32_t *perm, SahTree tr,
                                                      const uint32_t *root_nat_p, uint32_t leaf_size) {
    constexpr int W = kBlock / kWave;
    __shared__ float4 s_a[W][kSahSmall], s_b[W][kSahSmall];
    __shared__ unsigned long long s_key[W][kSahSmall];
    const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const uint32_t nsmall = min(*small_count, small_cap);
    for (uint32_t t = blockIdx.x * W + w; t < nsmall; t += gridDim.x * W) {
        const SahTask tk = small[t];
        const bool root_task = tk.parent < 0;
        uint32_t root_nat = root_task ? 0u : *root_nat_p;
        float4 *const va = s_a[w], *const vb = s_b[w];
        unsigned long long *const keys = s_key[w];
        uint32_t prim = 0;
        float4 lo = make_float4(0.0f, 0.0f, 0.0f, 0.0f), hi = lo;
        if ((uint32_t)lane < tk.count) {
            prim = perm[tk.first + lane];
            const Box b = pbox[prim];
            lo = b.lo;
            hi = b.hi;
        }
        // the lane's node: its lanes, parent and side
        uint32_t sf = 0, sc = (uint32_t)lane < tk.count ? tk.count : 0u, sd = tk.side;
        int32_t par = tk.parent;
        const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
        while (__builtin_amdgcn_ballot_w64(sc >= 2) != 0) {
            const bool act = sc >= 2;
            // a node of at most leaf_size primitives becomes one leaf whatever its
            // subtree: it is split at the index median without binning (no
            // reordering), so only the order inside the leaf differs from a full
            // SAH split
            const bool binned = act && sc > leaf_size;
            const uint32_t steps = wave_reduce<uint32_t>(binned ? sc : 0u, 0u,
                                                         [](uint32_t x, uint32_t y) { return max(x, y); });
            int axis = -1, bk = -1;
            uint32_t bins = 0;
            if (steps > 0) {
                float c[3], cl[3], ch[3];
                c[0] = 0.5f * lo.x + 0.5f * hi.x;  // as sah_centroid
                c[1] = 0.5f * lo.y + 0.5f * hi.y;
                c[2] = 0.5f * lo.z + 0.5f * hi.z;
                va[lane] = make_float4(c[0], c[1], c[2], 0.0f);
                keys[lane] = ~0ull;
                wave_sync();
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    cl[a] = INFINITY;
                    ch[a] = -INFINITY;
                }
                const uint32_t mine = binned ? sc : 0u;
                for (uint32_t j = 0; j < steps; j++) {
                    if (j >= mine) continue;
                    const float4 q = va[sf + j];
                    cl[0] = fminf(cl[0], q.x);
                    cl[1] = fminf(cl[1], q.y);
                    cl[2] = fminf(cl[2], q.z);
                    ch[0] = fmaxf(ch[0], q.x);
                    ch[1] = fmaxf(ch[1], q.y);
                    ch[2] = fmaxf(ch[2], q.z);
                }
                const SahFrame f = sah_frame(cl, ch);
#pragma unroll
                for (int a = 0; a < 3; a++)
                    if (f.ok(a)) bins |= (uint32_t)sah_bin(f, a, c[a]) << (8 * a);
                wave_sync();
                va[lane] = make_float4(lo.x, lo.y, lo.z, __uint_as_float(bins));
                vb[lane] = hi;
                wave_sync();
                // per axis: the union of the boxes up to the lane's bin and beyond it
                float l[3][6], r[3][6];
                uint32_t nleft[3] = {0, 0, 0};
#pragma unroll
                for (int a = 0; a < 3; a++)
#pragma unroll
                    for (int k = 0; k < 6; k++) l[a][k] = r[a][k] = k < 3 ? INFINITY : -INFINITY;
                for (uint32_t j = 0; j < steps; j++) {
                    if (j >= mine) continue;
                    const float4 p = va[sf + j], q = vb[sf + j];
                    const uint32_t pb = __float_as_uint(p.w);
                    const float v[6] = {p.x, p.y, p.z, q.x, q.y, q.z};
#pragma unroll
                    for (int a = 0; a < 3; a++) {
                        if (((pb >> (8 * a)) & 0xFFu) <= ((bins >> (8 * a)) & 0xFFu)) {
                            nleft[a]++;
#pragma unroll
                            for (int k = 0; k < 6; k++) l[a][k] = k < 3 ? fminf(l[a][k], v[k]) : fmaxf(l[a][k], v[k]);
                        } else {
#pragma unroll
                            for (int k = 0; k < 6; k++) r[a][k] = k < 3 ? fminf(r[a][k], v[k]) : fmaxf(r[a][k], v[k]);
                        }
                    }
                }
                // the node's cheapest split: lowest cost, then axis, then bin
                // (costs are not negative: their bits are in their order)
                unsigned long long key = ~0ull;
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    if (!f.ok(a) || nleft[a] == mine) continue;
                    const float cost =
                        half_area3(l[a][0], l[a][1], l[a][2], l[a][3], l[a][4], l[a][5]) * (float)nleft[a] +
                        half_area3(r[a][0], r[a][1], r[a][2], r[a][3], r[a][4], r[a][5]) * (float)(mine - nleft[a]);
                    if (!(cost < INFINITY)) continue;
                    const unsigned long long k = (unsigned long long)__float_as_uint(cost) << 32 |
                                                 (unsigned)(a << 8) | ((bins >> (8 * a)) & 0xFFu);
                    key = k < key ? k : key;
                }
                if (binned && key != ~0ull) atomicMin(&keys[sf], key);
                wave_sync();
                if (binned) {
                    key = keys[sf];
                    if (key != ~0ull) {
                        axis = (int)((key >> 8) & 3u);
                        bk = (int)(key & 0xFFu);
                    }
                }
            }
            const uint32_t pos = (uint32_t)lane - sf;
            const bool left = axis < 0 ? pos < sc / 2 : (int)((bins >> (8 * axis)) & 0xFFu) <= bk;
            const uint64_t seg = act ? (sc == 64u ? ~0ull : ((1ull << sc) - 1ull) << sf) : 0ull;
            const uint64_t lmask = __builtin_amdgcn_ballot_w64(act && left) & seg;
            const uint32_t nl = (uint32_t)__builtin_popcountll(lmask);
            const uint32_t m = tk.first + sf + nl;
            const bool is_root = root_task && par < 0;
            if (is_root) root_nat = m - 1;
            const uint32_t id = sah_node_id(m, is_root, root_nat);
            if (act && pos == 0)
                sah_write_node(tr, id, tk.first + sf, sc, axis < 0 ? 0 : axis, nl, par, sd);
            // stable partition
            if (steps > 0) {
                const uint32_t lrank = (uint32_t)__builtin_popcountll(lmask & below);
                const uint32_t dst = !act ? (uint32_t)lane : (left ? sf + lrank : sf + nl + (pos - lrank));
                va[dst] = make_float4(lo.x, lo.y, lo.z, __uint_as_float(prim));
                vb[dst] = hi;
                wave_sync();
                lo = va[lane];
                hi = vb[lane];
                prim = __float_as_uint(lo.w);
                wave_sync();
            }
            if (act) {
                par = (int32_t)id;
                sd = pos < nl ? 0u : 1u;
                sf = pos < nl ? sf : sf + nl;
                sc = pos < nl ? nl : sc - nl;
            }
        }
        if ((uint32_t)lane < tk.count) perm[tk.first + lane] = prim;
    }
}

__global__ void k_sah_init(uint32_t *ord, uint32_t *perm, uint32_t n, SahTask *task,
                           uint32_t *chunk, uint32_t *cstart, uint32_t *tc0, int *cb,
                           SahTask *small, uint32_t *nsmall, SahTask *mid, uint32_t *nmid) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) {
        ord[i] = i;
        perm[i] = i;
    }
    if (i == 0) {
        const SahTask root{0u, n, -1, 0u};
        if (n > kSahMid) {
            task[0] = root;
            tc0[0] = 0;
            sah_clear_bounds(cb);
        } else if (n > kSahSmall) {
            mid[0] = root;
            *nmid = 1;
        } else {
            small[0] = root;
            *nsmall = 1;
        }
    }
    const uint32_t nch = (n + kSahChunk - 1) / kSahChunk;
    if (n > kSahMid && i < nch) {
        chunk[i] = 0;
        cstart[i] = i * kSahChunk;
    }
}

__global__ void k_sah_publish(const uint32_t *src, uint32_t *dst, int k) {
    if (threadIdx.x == 0) {
        for (int i = 0; i < k; i++) dst[i] = src[i];
        __threadfence_system();
    }
}

// Host side of the binned-SAH topology: fills perm and the tree arrays.
int32_t sah_topology(const Box *pbox, uint32_t n, uint32_t *perm, SahTree tr, int leaf_size,
                     hipStream_t s) {
    if (n < 2) {
        if (n == 1) BVH_HIP_TRY(hipMemsetAsync(perm, 0, sizeof(uint32_t), s));
        return BVH_OK;
    }
    const uint32_t cap_task = n / (kSahMid + 1) + 1, cap_mid = n / (kSahSmall + 1) + 1;
    const uint32_t cap_small = n / 2 + 1;
    const uint32_t cap_chunk = (n + kSahChunk - 1) / kSahChunk + cap_task;
    uint32_t *ord[2], *ccnt, *cleft, *chunk[2], *cstart[2], *tc0[2], *counters, *small_count,
        *root_nat;
    SahTask *task[2], *small, *mid;
    SahSplit *split;
    int *cb[2], *bins, *cbins, *gbins;
    Arena ar;
    ar.request(&ord[0], n);
    ar.request(&ord[1], n);
    ar.request(&ccnt, (size_t)cap_chunk * kSahCounts);
    ar.request(&cleft, cap_chunk);
    ar.request(&task[0], cap_task);
    ar.request(&task[1], cap_task);
    ar.request(&chunk[0], cap_chunk);
    ar.request(&chunk[1], cap_chunk);
    ar.request(&cstart[0], cap_chunk);
    ar.request(&cstart[1], cap_chunk);
    ar.request(&split, cap_task);
    ar.request(&cb[0], (size_t)cap_task * 6);
    ar.request(&cb[1], (size_t)cap_task * 6);
    ar.request(&bins, (size_t)cap_task * kSahBinWords);
    ar.request(&cbins, (size_t)cap_chunk * kSahBinWords);
    ar.request(&gbins, (size_t)kMergeGroupTasks * kMergeGroups * kSahBinWords);
    ar.request(&tc0[0], cap_task);
    ar.request(&tc0[1], cap_task);
    ar.request(&small, cap_small);
    ar.request(&mid, cap_mid);
    ar.request(&counters, 2 * kSahMaxLevels + 4);
    BVH_TRY(ar.bind(s, kAreaSah));
    small_count = counters + 2 * kSahMaxLevels;
    root_nat = small_count + 1;
    uint32_t *err = small_count + 2, *mid_count = small_count + 3;
    BVH_HIP_TRY(hipMemsetAsync(counters, 0, (2 * kSahMaxLevels + 4) * sizeof(uint32_t), s));
    k_sah_init<<<grid_for(n), kBlock, 0, s>>>(ord[0], perm, n, task[0], chunk[0], cstart[0], tc0[0],
                                              cb[0], small, small_count, mid, mid_count);
    BVH_TRY(check_launch("sah init"));
    uint32_t *hw = host_words();
    if (!hw) return set_error(BVH_ENOMEM, "hipHostMalloc failed");
    volatile uint32_t *vw = hw + 8;
    uint32_t ntask = n > kSahMid ? 1u : 0u;
    uint32_t nchunk = (n + kSahChunk - 1) / kSahChunk;
    uint32_t nmid = n > kSahSmall && n <= kSahMid ? 1u : 0u;
    int cur = 0;
    if (ntask > 0) k_sah_bounds<<<nchunk, kBlock, 0, s>>>(n, pbox, cb[0]);
    for (int level = 0; ntask > 0; level++) {
        if (level >= kSahMaxLevels)
            return set_error(BVH_EUNSUPPORTED,
                             "bvh_build: SAH tree deeper than the traversal stack bound %d", kStackMax);
        // few tasks with several chunks each: merge them with several groups
        const uint32_t groups = (ntask <= kMergeGroupTasks && nchunk >= 2 * ntask) ? kMergeGroups : 1u;
        SahLevel lv{task[cur], chunk[cur], cstart[cur], cb[cur], bins, split, ntask, tc0[cur], cbins,
                    gbins, groups, ccnt, cleft};
        k_sah_bin<<<nchunk, kBlock, 0, s>>>(lv, ord[cur], pbox);
        if (nchunk > ntask) k_sah_merge<<<dim3(ntask, groups), kBlock, 0, s>>>(lv);
        const bool few = ntask <= kSplitFewTasks;
        const int threads = few ? kSplitFewThreads : kSplitManyThreads;
        (few ? k_sah_split<kSplitFewThreads> : k_sah_split<kSplitManyThreads>)<<<
            grid_for((uint64_t)ntask * kWave, threads), threads, 0, s>>>(
            lv, tr, root_nat, level == 0, task[cur ^ 1], chunk[cur ^ 1], cstart[cur ^ 1],
            tc0[cur ^ 1], cb[cur ^ 1], counters + 2 * level, small, small_count,
            mid, mid_count);
        vw[0] = vw[1] = vw[2] = kPending;
        k_sah_scatter<<<nchunk, kBlock, 0, s>>>(lv, ord[cur], pbox, ord[cur ^ 1], perm, cb[cur ^ 1],
                                                counters + 2 * level, mid_count, hw + 8, err);
        BVH_TRY(check_launch("sah level"));
        BVH_TRY(wait_host_word(vw, s, &ntask));
        BVH_TRY(wait_host_word(vw + 1, s, &nchunk));
        BVH_TRY(wait_host_word(vw + 2, s, &nmid));
        if (ntask > cap_task || nchunk > cap_chunk)
            return set_error(BVH_EHIP, "bvh_build: internal error (SAH task overflow)");
        cur ^= 1;
    }
    if (nmid > cap_mid) return set_error(BVH_EHIP, "bvh_build: internal error (SAH middle overflow)");
    if (nmid > 0)
        k_sah_mid<<<nmid, kMidThreads, 0, s>>>(mid, pbox, perm, tr, root_nat, small, small_count, err);
    // the device knows how many small tasks there are
    constexpr unsigned kSmallBlocks = 4096;
    k_sah_small<<<std::min(grid_for((uint64_t)cap_small * kWave), kSmallBlocks), kBlock, 0, s>>>(
        small, small_count, cap_small, pbox, perm, tr, root_nat, (uint32_t)leaf_size);
    vw[3] = kPending;
    k_sah_publish<<<1, 64, 0, s>>>(err, hw + 11, 1);
    BVH_TRY(check_launch("sah small nodes"));
    uint32_t bad = 0;
    BVH_TRY(wait_host_word(vw + 3, s, &bad));
    if (bad) return set_error(BVH_EHIP, "bvh_build: internal error (SAH partition)");
    return BVH_OK;
}

// a2, a3: Morton keys of the box centres, then a stable LSD radix sort of
// (key, primitive index), 8 bits per pass over the 3 * mbits key bits;
// returns which of the two buffers holds the sorted pairs.
template <typename KeyT>
int sort_morton(const Box *pbox, uint32_t n, const BuildInfo *info, int mbits, KeyT **keys,
                uint32_t **vals, uint32_t *hist, uint32_t nsort, hipStream_t s) {
    const uint32_t nhist = nsort * kRadix;
    k_morton<<<grid_for(n), kBlock, 0, s>>>(pbox, n, info, mbits, keys[0], vals[0]);
    int cur = 0;
    for (int shift = 0; shift < 3 * mbits; shift += 8) {
        k_radix_hist<<<nsort, kBlock, 0, s>>>(keys[cur], n, shift, hist, nsort);
        k_radix_offsets<<<kRadix, kBlock, 0, s>>>(hist, nsort, hist + nhist);
        k_radix_scatter<<<nsort, kBlock, 0, s>>>(keys[cur], vals[cur], keys[cur ^ 1],
                                                 vals[cur ^ 1], n, shift, hist, hist + nhist,
                                                 nsort);
        cur ^= 1;
    }
    return cur;
}

int32_t build_impl(const float *verts, int64_t n_verts, const int32_t *tris, int64_t n_tris,
                   bvh_handle_s *h, hipStream_t s) {
    const int n = (int)n_tris;
    const int L = h->leaf_size;

    Box *pbox, *nbox;
    float *partial;
    BuildInfo *info;
    uint64_t *keys[2];
    uint32_t *vals[2], *hist, *tile, *ifirst, *icount, *mark;
    int32_t *ileft, *iright, *parent;
    uint8_t *iaxis;
    const uint32_t nb = grid_for(n);
    const uint32_t nsort = (uint32_t)((n + kSortTile - 1) / kSortTile);
    const uint32_t nhist = nsort * kRadix;
    const uint32_t max_scan = std::max<uint32_t>(nhist, (uint32_t)n);
    const int nblocks = (n + kRangeBlock - 1) / kRangeBlock;
    int levels = 1;
    while ((1 << levels) <= nblocks) levels++;
    Box *table, *pre, *suf;
    float *area;
    Arena arena;
    arena.request(&pbox, n);
    arena.request(&partial, (size_t)nb * 12);
    arena.request(&info, 1);
    arena.request(&keys[0], n);
    arena.request(&keys[1], n);
    arena.request(&vals[0], n);
    arena.request(&vals[1], n);
    arena.request(&hist, nhist + kRadix);  // counts, then the digit totals
    arena.request(&tile, (max_scan + kScanTile - 1) / kScanTile + 1);
    arena.request(&ileft, n - 1);
    arena.request(&iright, n - 1);
    arena.request(&ifirst, n - 1);
    arena.request(&icount, n - 1);
    arena.request(&iaxis, n - 1);
    arena.request(&parent, 2 * (size_t)n - 1);
    arena.request(&nbox, 2 * (size_t)n - 1);
    arena.request(&mark, n);
    arena.request(&table, (size_t)levels * nblocks);
    arena.request(&pre, n);
    arena.request(&suf, n);
    arena.request(&area, n - 1);
    uint32_t *bound_slots;
    arena.request(&bound_slots, 3 * kMaxSlots * kSlotStride);  // stack, depth, leaf-count slots
    int32_t *cand_all = nullptr;  // wide layouts: the child list of every binary node
    uint32_t *ni_all = nullptr;
    if (layout_arity(h->layout) > 2) {
        const size_t m = (size_t)std::max(1, n - 1);
        arena.request(&cand_all, m * (size_t)layout_arity(h->layout));
        arena.request(&ni_all, m);
    }
    BVH_TRY(arena.bind(s, kAreaBuild));

    const bool wide = h->layout == BVH_LAYOUT_BVH4 || h->layout == BVH_LAYOUT_BVH8_Q8 ||
                      h->layout == BVH_LAYOUT_BVH8_Q16;
    {
        // k_karras writes the parent of every node (the root's too) when n > 1
        const uint32_t nslots = 3 * kMaxSlots * kSlotStride;
        const uint32_t nmark = wide ? 0u : (uint32_t)n;
        const uint64_t nparent =
            (h->builder == BVH_BUILDER_SAH || n == 1) ? 2 * (uint64_t)n - 1 : 0u;
        const uint64_t m = std::max<uint64_t>(std::max<uint64_t>(nslots, nmark), nparent);
        k_build_init<<<grid_for(m), kBlock, 0, s>>>(info, bound_slots, nslots, mark, nmark, parent,
                                                    nparent);
    }

    // a1, a2
    const uint32_t nbp = (uint32_t)(((uint64_t)n + kPrimItems * kBlock - 1) / (kPrimItems * kBlock));
    k_prim_bounds<<<nbp, kBlock, 0, s>>>(verts, n_verts, tris, n, pbox, partial, info);
    const bool small = h->builder == BVH_BUILDER_LBVH && (uint32_t)n <= kSmallMax;
    if (!small) k_bounds_final<<<1, kBlock, 0, s>>>(partial, nbp, info);
    const uint32_t *perm = nullptr;
    SideStream *side = nullptr;
    // a8 leaf data for the wide layouts, queued as soon as the order is final,
    // on the side stream: the leaf block's hipMalloc (and the node block's,
    // from the hint) block the host while the queued kernels run, then the
    // leaf kernel overlaps the hierarchy kernels
    // the point of the stream after which the sorted order is final: the
    // side stream's leaf data waits for it (and not for the kernels queued
    // on the build stream after it)
    bool sorted_marked = false;
    auto mark_sorted = [&]() -> int32_t {
        if (!wide || sorted_marked) return BVH_OK;
        sorted_marked = true;
        side = side_stream(h->device);
        if (side) BVH_HIP_TRY(hipEventRecord(side->ready, s));
        return BVH_OK;
    };
    auto leaf_data_early = [&]() -> int32_t {
        if (!wide) return BVH_OK;
        BVH_TRY(mark_sorted());
        BVH_TRY(alloc_leaf_block(h));
        BVH_TRY(alloc_node_block_ahead(h));
        const LeafSource early{verts, n_verts, tris, perm, (uint32_t)n};
        if (!side) return emit_leaf_data(h, early, s);
        BVH_HIP_TRY(hipStreamWaitEvent(side->stream, side->ready, 0));
        BVH_TRY(emit_leaf_data(h, early, side->stream));
        BVH_HIP_TRY(hipEventRecord(side->done, side->stream));
        return BVH_OK;
    };
    uint32_t *hw = host_words();
    if (!hw) return set_error(BVH_ENOMEM, "hipHostMalloc failed");
    volatile uint32_t *nleaf_word = hw + 8;
    *nleaf_word = kPending;
    bool leaves_told = false;  // a queued kernel already writes the leaf count there
    uint32_t *karras_leaves = nullptr;  // leaf-count slots filled by k_karras (else by k_count_leaves)
    if (h->builder == BVH_BUILDER_SAH) {
        // a4 alternative: binned-SAH topology over the primitive boxes
        BVH_TRY(check_launch("bounds"));
        SahTree tr{ileft, iright, parent, ifirst, icount, iaxis, n};
        BVH_TRY(sah_topology(pbox, (uint32_t)n, vals[0], tr, L, s));
        perm = vals[0];
        BVH_TRY(leaf_data_early());
    } else if (small) {
        // a2, a3, a4 in one launch; at most 3 * 8 key bits at this size
        uint32_t *leaf_word = wide && n > 1 ? hw + 8 : nullptr;
        k_small_hierarchy<<<1, kSmallThreads, 0, s>>>(pbox, (uint32_t)n, partial, nbp, info,
                                                      morton_bits(n), vals[0], ileft, iright, ifirst,
                                                      icount, iaxis, parent, L, leaf_word);
        leaves_told = leaf_word != nullptr;
        BVH_TRY(check_launch("small hierarchy"));
        perm = vals[0];
        BVH_TRY(leaf_data_early());
    } else {
        // a2, a3: keys of 3 * mbits bits, in 32-bit words when they fit
        // (the key buffers hold 64-bit words either way)
        const int mbits = morton_bits(n);
        const bool narrow = 3 * mbits <= 32;
        uint32_t *k32[2] = {reinterpret_cast<uint32_t *>(keys[0]),
                            reinterpret_cast<uint32_t *>(keys[1])};
        int cur = 0;
        if (narrow)
            cur = sort_morton(pbox, (uint32_t)n, info, mbits, k32, vals, hist, nsort, s);
        else
            cur = sort_morton(pbox, (uint32_t)n, info, mbits, keys, vals, hist, nsort, s);
        BVH_TRY(check_launch("morton/radix sort"));
        perm = vals[cur];
        BVH_TRY(mark_sorted());

        // a4 (for the wide layouts, also the leaf count of the collapse),
        // queued before the leaf data's allocations so that the GPU does not
        // wait for them
        if (n > 1) {
            karras_leaves = wide ? bound_slots + 2 * kMaxSlots * kSlotStride : nullptr;
            if (narrow)
                k_karras<<<grid_for(n - 1), kBlock, 0, s>>>(k32[cur], n, ileft, iright, ifirst,
                                                            icount, iaxis, parent, L, karras_leaves);
            else
                k_karras<<<grid_for(n - 1), kBlock, 0, s>>>(keys[cur], n, ileft, iright, ifirst,
                                                            icount, iaxis, parent, L, karras_leaves);
        }
        BVH_TRY(leaf_data_early());
    }
    {  // a5
        k_leaf_boxes<<<nb, kBlock, 0, s>>>(pbox, perm, n, nbox, table, pre, suf);
        for (int k = 1; k < levels; k += 3)
            k_table_levels<<<grid_for(nblocks), kBlock, 0, s>>>(table, nblocks, k,
                                                                std::min(3, levels - k));
        if (n > 1)
            k_internal_boxes<<<grid_for(n - 1), kBlock, 0, s>>>(ifirst, icount, n, table, nblocks,
                                                                pre, suf, nbox, area);
    }
    BVH_TRY(check_launch("hierarchy/boxes"));
    // a6
    TreeView tv{n, L, ileft, iright, parent, ifirst, icount, iaxis, nbox, area, bound_slots,
                bound_slots + kMaxSlots * kSlotStride};
    // the wide layouts read the leaf count from a host-mapped word instead of
    // draining the stream (and need no leaf marks); the others need the scene
    // box and the marks' exclusive scan before packing
    if (wide && !leaves_told) {
        uint32_t *leaf_slots = bound_slots + 2 * kMaxSlots * kSlotStride;
        if (!karras_leaves)
            k_count_leaves<<<grid_for(2 * (uint64_t)n - 1), kBlock, 0, s>>>(tv, leaf_slots);
        *nleaf_word = kPending;  // the SAH build has used the word
        k_fold_leaf_count<<<1, kBlock, 0, s>>>(leaf_slots, hw + 8);
    } else if (!wide) {
        k_mark_leaves<<<grid_for(2 * (uint64_t)n - 1), kBlock, 0, s>>>(tv, mark);
        scan_u32(mark, mark, n, tile, &info->n_leaves, s);
    }
    BVH_TRY(check_launch("collapse"));
    BuildInfo hi;
    BuildInfo *pin = pinned_scratch<BuildInfo>();
    if (!pin) return set_error(BVH_ENOMEM, "hipHostMalloc failed");
    const LeafSource ls{verts, n_verts, tris, perm, (uint32_t)n};
    if (!wide) {
        BVH_HIP_TRY(hipMemcpyAsync(pin, info, sizeof(hi), hipMemcpyDeviceToHost, s));
        BVH_TRY(alloc_leaf_block(h));  // while the queued kernels run
        BVH_HIP_TRY(hipStreamSynchronize(s));
        hi = *pin;
        if (hi.err & 1u) return set_error(BVH_EINVAL, "bvh_build: a vertex index is outside [0, n_verts)");
        for (int a = 0; a < 3; a++) {
            h->scene_lo[a] = hi.slo[a];
            h->scene_hi[a] = hi.shi[a];
        }
        h->n_leaves = hi.n_leaves;
    }

    // a7
    if (h->layout == BVH_LAYOUT_AABB2) {
        h->n_nodes = 2 * (int64_t)hi.n_leaves - 1;
        BVH_TRY(emit_leaf_data(h, ls, s));
        BVH_TRY(alloc_node_block(h, h->n_nodes));
        k_emit_aabb2<<<grid_for(2 * (uint64_t)n - 1), kBlock, 0, s>>>(
            tv, mark, static_cast<bvh_node_aabb2 *>(h->nodes), (uint32_t)h->n_nodes, info);
        BVH_TRY(check_launch("aabb2 packing"));
    } else if (h->layout == BVH_LAYOUT_PBRT_SOAOS) {
        // the AABB2 records, split into a box array and a topology array
        h->n_nodes = 2 * (int64_t)hi.n_leaves - 1;
        Arena ar;
        bvh_node_aabb2 *tmp = nullptr;
        ar.request(&tmp, (size_t)h->n_nodes);
        BVH_TRY(ar.bind(s, kAreaBuildWide));
        BVH_TRY(emit_leaf_data(h, ls, s));
        BVH_TRY(alloc_node_block(h, h->n_nodes));
        k_emit_aabb2<<<grid_for(2 * (uint64_t)n - 1), kBlock, 0, s>>>(tv, mark, tmp,
                                                                      (uint32_t)h->n_nodes, info);
        k_split_aabb2<<<grid_for((uint64_t)h->n_nodes), kBlock, 0, s>>>(
            tmp, (uint32_t)h->n_nodes, static_cast<bvh_node_box_f32 *>(h->nodes),
            const_cast<bvh_node_topo *>(static_cast<const bvh_node_topo *>(
                topo_of(h->nodes, h->n_nodes, h->layout))));
        BVH_TRY(check_launch("pbrt-soaos packing"));
    } else if (h->layout == BVH_LAYOUT_SHARED_SLAB) {
        // the AABB2 tree with one slab per node in place of its box
        h->n_nodes = 2 * (int64_t)hi.n_leaves - 1;
        Arena ar;
        bvh_node_aabb2 *tmp = nullptr;
        ar.request(&tmp, (size_t)h->n_nodes);
        BVH_TRY(ar.bind(s, kAreaBuildWide));
        BVH_TRY(emit_leaf_data(h, ls, s));
        BVH_TRY(alloc_node_block(h, h->n_nodes));
        k_emit_aabb2<<<grid_for(2 * (uint64_t)n - 1), kBlock, 0, s>>>(tv, mark, tmp,
                                                                      (uint32_t)h->n_nodes, info);
        k_pack_slab<<<grid_for((uint64_t)h->n_nodes), kBlock, 0, s>>>(
            tmp, (uint32_t)h->n_nodes, info, static_cast<bvh_node_slab *>(h->nodes));
        BVH_TRY(check_launch("shared-slab packing"));
    } else if (layout_scene_frame(h->layout)) {
        // the AABB2 tree, re-encoded node by node in the scene frame
        const bool pq = !layout_sg_eq(h->layout);
        h->n_nodes = 2 * (int64_t)hi.n_leaves - 1;
        const WorldFrame fr = world_frame(hi.slo, hi.shi, pq ? 65535.0f : 1023.0f);
        for (int a = 0; a < 3; a++) {
            h->frame_origin[a] = fr.o[a];
            h->frame_scale[a] = fr.s[a];
            h->frame_top[a] = pq ? 0.0f : fr.top[a];
        }
        Arena ar;
        bvh_node_aabb2 *tmp = nullptr;
        ar.request(&tmp, (size_t)h->n_nodes);
        BVH_TRY(ar.bind(s, kAreaBuildWide));
        BVH_TRY(emit_leaf_data(h, ls, s));
        BVH_TRY(alloc_node_block(h, h->n_nodes));
        k_emit_aabb2<<<grid_for(2 * (uint64_t)n - 1), kBlock, 0, s>>>(tv, mark, tmp,
                                                                      (uint32_t)h->n_nodes, info);
        const unsigned g = grid_for((uint64_t)h->n_nodes);
        const uint32_t nn = (uint32_t)h->n_nodes;
        if (h->layout == BVH_LAYOUT_PBRT_Q16)
            k_pack_pbrt_q16<false><<<g, kBlock, 0, s>>>(
                tmp, nn, fr, static_cast<bvh_node_pbrt_q16 *>(h->nodes), nullptr, nullptr, info);
        else if (h->layout == BVH_LAYOUT_PBRT_Q16_SOAOS)
            k_pack_pbrt_q16<true><<<g, kBlock, 0, s>>>(
                tmp, nn, fr, nullptr, static_cast<bvh_node_box_q16 *>(h->nodes),
                static_cast<uint32_t *>(const_cast<void *>(topo_of(h->nodes, h->n_nodes, h->layout))),
                info);
        else if (h->layout == BVH_LAYOUT_SG_EQ)
            k_pack_sg_eq<false><<<g, kBlock, 0, s>>>(tmp, nn, fr, h->nodes, info);
        else
            k_pack_sg_eq<true><<<g, kBlock, 0, s>>>(tmp, nn, fr, h->nodes, info);
        BVH_TRY(check_launch("scene-frame packing"));
    } else if (h->layout == BVH_LAYOUT_BVH4) {
        BVH_TRY(pack_wide<BVH_LAYOUT_BVH4>(tv, nleaf_word, cand_all, ni_all, info, h, ls, s));
    } else if (h->layout == BVH_LAYOUT_BVH8_Q8) {
        BVH_TRY(pack_wide<BVH_LAYOUT_BVH8_Q8>(tv, nleaf_word, cand_all, ni_all, info, h, ls, s));
    } else {
        BVH_TRY(pack_wide<BVH_LAYOUT_BVH8_Q16>(tv, nleaf_word, cand_all, ni_all, info, h, ls, s));
    }
    if (!wide) {  // pack_wide folds them itself
        k_fold_max_slots<<<1, kBlock, 0, s>>>(tv.stack_slots, tv.depth_slots, info);
        BVH_TRY(check_launch("stack bound"));
    }
    if (side) BVH_HIP_TRY(hipStreamWaitEvent(s, side->done, 0));  // the leaf data is part of the build
    BVH_HIP_TRY(hipMemcpyAsync(pin, info, sizeof(hi), hipMemcpyDeviceToHost, s));
    BVH_HIP_TRY(hipStreamSynchronize(s));
    hi = *pin;
    if (wide) {
        if (hi.err & 1u) return set_error(BVH_EINVAL, "bvh_build: a vertex index is outside [0, n_verts)");
        for (int a = 0; a < 3; a++) {
            h->scene_lo[a] = hi.slo[a];
            h->scene_hi[a] = hi.shi[a];
        }
    }
    if (hi.err & 4u) return set_error(BVH_EHIP, "bvh_build: internal error (malformed hierarchy)");
    if (hi.err & 2u)
        return set_error(BVH_EUNSUPPORTED, "bvh_build: non-finite box extent (coordinates too large?)");
    h->depth = (int32_t)hi.max_depth;
    h->max_stack = (int32_t)hi.max_stack;
    if (h->max_stack > kStackMax)
        return set_error(BVH_EUNSUPPORTED, "bvh_build: traversal stack bound %d exceeds %d",
                         h->max_stack, kStackMax);
    return BVH_OK;
}

}  // namespace
}  // namespace bvhlib

using namespace bvhlib;

namespace bvhlib {

int32_t build_handle(const float *verts, int64_t n_verts, const int32_t *tris, int64_t n_tris,
                     int32_t layout, int32_t leaf_size, int32_t leaf_mode, int32_t stack_lds,
                     int32_t builder, hipStream_t s, bvh_handle_s **out) {
    *out = nullptr;
    BVH_TRY(require_device());
    int dev = 0;
    BVH_HIP_TRY(hipGetDevice(&dev));
    bvh_handle_s *h = new bvh_handle_s;
    h->device = dev;
    h->layout = layout;
    h->leaf_mode = leaf_mode;
    h->leaf_size = leaf_size;
    h->stack_lds = stack_lds;
    h->builder = builder;
    h->arity = layout_arity(layout);
    h->n_tris = n_tris;
    h->n_verts = n_verts;
    h->node_bytes = node_record_bytes(layout);
    if (n_tris == 0) {
        *out = h;
        return BVH_OK;
    }
    int32_t rc = build_impl(verts, n_verts, tris, n_tris, h, s);
    if (rc != BVH_OK) {
        std::string msg = bvh_last_error();
        bvh_destroy(h);
        return set_error(rc, "%s", msg.c_str());
    }
    *out = h;
    return BVH_OK;
}

}  // namespace bvhlib

extern "C" int32_t bvh_build(const float *verts, int64_t n_verts, const int32_t *tris,
                             int64_t n_tris, int32_t layout, const bvh_build_opts *opts,
                             void *stream, bvh_handle_t *out) {
    if (!out) return set_error(BVH_EINVAL, "bvh_build: out is null");
    *out = nullptr;
    if (n_tris < 0 || n_verts < 0) return set_error(BVH_EINVAL, "bvh_build: negative size");
    if (n_tris > 0 && (!verts || !tris)) return set_error(BVH_EINVAL, "bvh_build: null mesh pointer");
    if (n_tris > 0 && n_verts == 0) return set_error(BVH_EINVAL, "bvh_build: triangles without vertices");
    if (layout < 0 || layout >= BVH_NUM_LAYOUTS)
        return set_error(BVH_EINVAL, "bvh_build: unknown layout %d", layout);
    // LDS stack default: binary trees push one entry per level (32 entries of
    // 4 B); wide trees push up to arity-1 entries of 8 B (16 entries)
    int32_t leaf_size = 4, leaf_mode = BVH_LEAF_COMPACT;
    int32_t stack_lds = layout_arity(layout) == 2 ? 32 : 16;
    int32_t builder = BVH_BUILDER_LBVH;
    if (opts) {
        for (int k = 0; k < 4; k++)
            if (opts->reserved[k] != 0) return set_error(BVH_EINVAL, "bvh_build: reserved option set");
        if (opts->leaf_size != 0) leaf_size = opts->leaf_size;
        if (opts->leaf_mode != 0) leaf_mode = opts->leaf_mode;
        if (opts->stack_lds != 0) stack_lds = opts->stack_lds;
        builder = opts->builder;
    }
    if (builder != BVH_BUILDER_LBVH && builder != BVH_BUILDER_SAH)
        return set_error(BVH_EINVAL, "bvh_build: unknown builder %d", builder);
    const int32_t max_leaf =  // the scene-frame binary layouts store a u4 count
        layout_scene_frame(layout) ? 15 : kMaxLeafSize;
    if (leaf_size < 1 || leaf_size > max_leaf)
        return set_error(BVH_EINVAL, "bvh_build: leaf_size %d outside 1..%d", leaf_size, max_leaf);
    if (leaf_mode != BVH_LEAF_COMPACT && leaf_mode != BVH_LEAF_INDEXED)
        return set_error(BVH_EINVAL, "bvh_build: unknown leaf mode %d", leaf_mode);
    if (stack_lds != 8 && stack_lds != 16 && stack_lds != 32)
        return set_error(BVH_EINVAL, "bvh_build: stack_lds %d is not 8, 16 or 32", stack_lds);
    if (n_tris > kMaxTris)
        return set_error(BVH_EUNSUPPORTED, "bvh_build: %lld triangles exceed %lld",
                         (long long)n_tris, (long long)kMaxTris);
    return build_handle(verts, n_verts, tris, n_tris, layout, leaf_size, leaf_mode, stack_lds,
                        builder, static_cast<hipStream_t>(stream), out);
}
