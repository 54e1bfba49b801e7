// The library's pool of released device blocks (workspace.hip, compiled for
// the host) over a stand-in for the runtime's allocator with a byte budget per
// device.  Built and run by test_block_pool.py; prints one line per check.
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <map>

#include "internal.h"

namespace {
std::map<void *, std::pair<int, size_t>> g_live;
std::map<int, size_t> g_used;
size_t g_budget = 0;
int g_device = 0;
hipError_t g_last = hipSuccess;
}  // namespace

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
    if (g_used[g_device] + bytes > g_budget) return g_last = hipErrorOutOfMemory;
    *p = std::malloc(1);
    g_live[*p] = {g_device, bytes};
    g_used[g_device] += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto it = g_live.find(p);
    if (it == g_live.end()) return hipErrorInvalidValue;
    g_used[it->second.first] -= it->second.second;
    g_live.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetLastError(void) {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int *d) { *d = g_device; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

namespace bvhlib {
int32_t set_error(int32_t code, const char *, ...) { return code; }
}  // namespace bvhlib

using namespace bvhlib;

int main() {
    constexpr size_t MB = size_t(1) << 20;
    DeviceBlock b, c;
    // an allocation of any kind gets the memory of the idle blocks
    g_budget = 1000 * MB;
    block_alloc(0, 400 * MB, &b);
    block_release(0, &b);
    void *p = nullptr;
    std::printf("kept %zu\n", g_used[0] / MB);
    const hipError_t got = device_malloc(0, 900 * MB, &p);
    std::printf("malloc %d used %zu\n", (int)got, g_used[0] / MB);
    const hipError_t not_got = device_malloc(0, 200 * MB, &p);
    std::printf("refused %d null %d last %d\n", (int)not_got, p == nullptr, (int)hipGetLastError());
    (void)hipFree(g_live.begin()->first);

    // a device's blocks are aged by its own releases only
    g_budget = 100000 * MB;
    g_device = 1;
    block_alloc(1, 40 * MB, &b);
    block_release(1, &b);
    g_device = 0;
    for (int i = 0; i < 200; i++) {
        block_alloc(0, 10 * MB, &c);
        block_release(0, &c);
    }
    g_device = 1;
    block_alloc(1, 10 * MB, &c);
    block_release(1, &c);
    std::printf("ages %zu %zu\n", g_used[0] / MB, g_used[1] / MB);
    for (int i = 0; i < 200; i++) {
        block_alloc(1, 10 * MB, &c);
        block_release(1, &c);
    }
    std::printf("aged %zu %zu\n", g_used[0] / MB, g_used[1] / MB);
    block_trim(0);
    std::printf("trimmed %zu %zu\n", g_used[0] / MB, g_used[1] / MB);
    return 0;
}
