// The library's device memory pool (memory.hip) over a stand-in for the runtime: devices of a given
// size, whose allocations are counted.  Prints "ok" or the check that failed.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <thread>

#include "memory.hpp"

namespace {
std::mutex g_lock;
std::map<void*, std::pair<int, size_t>> g_held;   // device, bytes
size_t g_total = (size_t)16 << 30;
int g_device = 0;
bool g_full = false;   // allocations fail until something is freed

size_t held(int device) {
    std::lock_guard<std::mutex> hold(g_lock);
    size_t n = 0;
    for (auto& h : g_held) n += h.second.first == device ? h.second.second : 0;
    return n;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) {
    *d = g_device;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceTotalMem(size_t* n, hipDevice_t) {
    *n = g_total;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> hold(g_lock);
    if (g_full) return hipErrorOutOfMemory;
    *p = std::malloc(16);
    g_held[*p] = {g_device, n};
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    std::lock_guard<std::mutex> hold(g_lock);
    if (!g_held.erase(p)) std::abort();
    g_full = false;
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
}

#define CHECK(x)                                                  \
    do {                                                          \
        if (!(x)) {                                               \
            std::printf("%s (line %d)\n", #x, __LINE__);          \
            return 1;                                             \
        }                                                         \
    } while (0)

using namespace cuesim;

int main() {
    const size_t G = (size_t)1 << 30, M = (size_t)1 << 20;
    void* p[64] = {};
    // while an object lives, a sixteenth of each device's memory
    device_memory_user(1);
    for (int device : {0, 1}) {
        g_device = device;
        for (int k = 0; k < 24; ++k) CHECK(device_malloc(&p[k], 200 * M + k) == hipSuccess);
        for (int k = 0; k < 24; ++k) device_free(p[k]);
        CHECK(held(device) <= g_total / 16 && held(device) > g_total / 16 - 201 * M);
        CHECK(device_idle_bytes(device) == held(device));
    }
    // a block larger than that is not kept; one of nearly its size is reused
    CHECK(device_malloc(&p[0], 2 * G) == hipSuccess);
    device_free(p[0]);
    CHECK(held(1) <= g_total / 16);
    CHECK(device_malloc(&p[0], 100 * M) == hipSuccess);
    device_free(p[0]);
    CHECK(device_malloc(&p[1], 99 * M) == hipSuccess && p[1] == p[0]);
    device_free(p[1]);
    // between objects, no more than a sixteenth nor 1 GiB, on every device
    device_memory_user(-1);
    for (int device : {0, 1}) CHECK(held(device) <= G);
    // the next object: what is idle serves it; when the device is full it is all given back first
    device_memory_user(1);
    g_device = 0;
    g_full = true;
    CHECK(device_malloc(&p[0], 3 * G) == hipSuccess);
    CHECK(held(0) == 3 * G && device_idle_bytes(0) == 0 && device_idle_bytes(1) == held(1));
    g_full = true;
    CHECK(device_malloc(&p[1], G) == hipErrorOutOfMemory);
    g_full = false;
    // everything idle back on request, with an object alive; what is in use stays
    CHECK(device_malloc(&p[1], 64 * M) == hipSuccess);
    device_free(p[1]);
    CHECK(device_idle_bytes(0) == 64 * M);
    CHECK(release_device_memory() == hipSuccess);
    CHECK(held(0) == 3 * G && held(1) == 0 && device_idle_bytes(0) == 0);
    device_free(p[0]);
    device_memory_user(-1);
    CHECK(release_device_memory() == hipSuccess && held(0) == 0);
    // several threads
    device_memory_user(1);
    std::thread t[6];
    for (int k = 0; k < 6; ++k)
        t[k] = std::thread([k, M] {
            void* q[5];
            for (int r = 0; r < 400; ++r) {
                for (int i = 0; i < 5; ++i)
                    if (device_malloc(&q[i], (1 + (k + r + i) % 7) * 40 * M) != hipSuccess)
                        std::abort();
                for (int i = 0; i < 5; ++i) device_free(q[i]);
                if (r % 50 == 49 && release_device_memory() != hipSuccess) std::abort();
            }
        });
    for (auto& x : t) x.join();
    CHECK(held(0) == device_idle_bytes(0) && held(0) <= g_total / 16);
    // host flags: words and events of their own, zeroed again, of the device asked for
    HostFlag f[130];
    for (int k = 0; k < 130; ++k) {
        CHECK(host_flag(&f[k]) == hipSuccess && *f[k].word == 0 && f[k].device == 0);
        for (int i = 0; i < k; ++i) CHECK(f[k].word != f[i].word && f[k].event != f[i].event);
    }
    *f[5].word = 7;
    host_flag_free(f[5]);
    host_flag_free(HostFlag{});
    g_device = 1;
    HostFlag other;
    CHECK(host_flag(&other) == hipSuccess && other.device == 1 && other.event != f[5].event);
    g_device = 0;
    const HostFlag before = f[5];
    CHECK(host_flag(&f[5]) == hipSuccess && f[5].word == before.word && *f[5].word == 0 &&
          f[5].event == before.event);
    std::printf("ok\n");
    return 0;
}
