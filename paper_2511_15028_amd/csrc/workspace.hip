// Grow-only device work areas, one per (device, stream, purpose), kept until
// the process ends.  Builds and traces on one stream are ordered by that
// stream, so they can reuse its area; work on different streams gets
// different areas.  In steady state no call allocates or frees device memory
// (stream-ordered frees cost up to milliseconds each on this platform).
#include <list>
#include <map>
#include <mutex>
#include <tuple>

#include "internal.h"

namespace bvhlib {
namespace {

struct Area {
    void *ptr = nullptr;
    size_t bytes = 0;
};

std::mutex g_mutex;
std::map<std::tuple<int, hipStream_t, int>, Area> g_areas;

// Device blocks of destroyed handles, kept for the next builds.  Rebuilding a
// moving scene every frame otherwise pays a hipFree (with the GPU idle) and a
// hipMalloc per block and frame: build, two traces and release of 2.1 M
// triangles 1,800 us a frame, with the blocks kept 1,370 us; of 1,024 triangles
// 197 and 181 us.
//
// Bounded: kPoolBlocks blocks and kPoolBytes bytes per device, the longest idle
// one freed first; a block that kPoolAge of its device's releases have passed by
// is freed too, and so is every block before the library reports an allocation
// failure, and on bvh_trim.
// Safe with any threads and streams: a block enters the pool only once its
// device is idle (block_release's contract), so whoever takes it next, on any
// stream, finds no work using it.
constexpr size_t kPoolBlocks = 8;
constexpr size_t kPoolBytes = size_t(512) << 20;
constexpr uint64_t kPoolAge = 64;

struct IdleBlock {
    int device;
    DeviceBlock block;
    uint64_t since;  // its device's releases when it came in
};

std::mutex g_pool_mutex;
std::list<IdleBlock> g_idle;             // oldest first
std::map<int, uint64_t> g_releases;      // per device

}  // namespace

void block_trim(int device) {
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    for (auto it = g_idle.begin(); it != g_idle.end();) {
        if (it->device != device) {
            ++it;
            continue;
        }
        (void)hipFree(it->block.ptr);
        it = g_idle.erase(it);
    }
}

hipError_t device_malloc(int device, size_t bytes, void **out) {
    hipError_t e = hipMalloc(out, bytes);
    if (e != hipSuccess) {  // the idle blocks may be what is missing
        (void)hipGetLastError();
        block_trim(device);
        e = hipMalloc(out, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *out = nullptr;
    }
    return e;
}

// A block of at least `bytes` on `device` (the current device), idle.
hipError_t block_alloc(int device, size_t bytes, DeviceBlock *out) {
    {
        std::lock_guard<std::mutex> lock(g_pool_mutex);
        // the smallest that fits and is not more than a quarter too large
        auto best = g_idle.end();
        for (auto it = g_idle.begin(); it != g_idle.end(); ++it)
            if (it->device == device && it->block.bytes >= bytes && it->block.bytes <= bytes + bytes / 4 &&
                (best == g_idle.end() || it->block.bytes < best->block.bytes))
                best = it;
        if (best != g_idle.end()) {
            *out = best->block;
            g_idle.erase(best);
            return hipSuccess;
        }
    }
    void *p = nullptr;
    const hipError_t e = device_malloc(device, bytes, &p);
    *out = e == hipSuccess ? DeviceBlock{p, bytes} : DeviceBlock{};
    return e;
}

// Gives a block back.  No work that uses it is queued or running any more, and
// its device is the current one.
void block_release(int device, DeviceBlock *b) {
    if (!b->ptr) return;
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    const DeviceBlock given = *b;
    *b = DeviceBlock{};
    uint64_t now = 0;
    try {
        now = ++g_releases[device];
        g_idle.push_back(IdleBlock{device, given, now});
    } catch (...) {  // no host memory to remember it with
        (void)hipFree(given.ptr);
        return;
    }
    size_t blocks = 0, bytes = 0;
    for (auto it = g_idle.end(); it != g_idle.begin();) {  // newest first
        --it;
        if (it->device != device) continue;
        blocks++;
        bytes += it->block.bytes;
        if (blocks > kPoolBlocks || bytes > kPoolBytes || now - it->since > kPoolAge) {
            bytes -= it->block.bytes;
            blocks--;
            (void)hipFree(it->block.ptr);
            it = g_idle.erase(it);
        }
    }
}

int32_t stream_workspace(hipStream_t s, int purpose, size_t bytes, void **out) {
    *out = nullptr;
    int dev = 0;
    BVH_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(g_mutex);
    Area &a = g_areas[std::make_tuple(dev, s, purpose)];
    if (a.bytes < bytes) {
        if (a.ptr) {
            // the old area may still be in use by queued work on this stream
            BVH_HIP_TRY(hipStreamSynchronize(s));
            BVH_HIP_TRY(hipFree(a.ptr));
            a.ptr = nullptr;
            a.bytes = 0;
        }
        const size_t grow = bytes + bytes / 4;  // headroom against repeated growth
        const hipError_t e = device_malloc(dev, grow, &a.ptr);
        if (e != hipSuccess)
            return set_error(BVH_ENOMEM, "work area of %zu bytes: %s", grow, hipGetErrorString(e));
        a.bytes = grow;
    }
    *out = a.ptr;
    return BVH_OK;
}

}  // namespace bvhlib
