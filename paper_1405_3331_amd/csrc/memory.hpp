// memory.hpp -- device memory of the library's objects.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <vector>

namespace cuesim {

// Device memory of at least `bytes` on the current device, from blocks that released objects
// left behind where one fits (up to a quarter larger), else from the runtime.  The contents
// are undefined.  Safe from several threads.
hipError_t device_malloc(void** p, size_t bytes);
// Give a block back.  All device work that uses it must have finished: the next owner may
// write it at once, on any stream.  nullptr is a no-op.
void device_free(void* p);
// Every idle block back to the runtime.
hipError_t release_device_memory();
// Bytes that idle blocks hold on a device (free memory that the runtime does not count).
size_t device_idle_bytes(int device);
// An object that owns device memory begins or ends; between objects fewer idle blocks are kept.
void device_memory_user(int change);

// A zeroed word of pinned host memory, a line of its own, and an event of the current device (without
// timing), which the library keeps for the next object when one gives them back: as many as objects
// lived at once.  (From the runtime a word takes longer than the rest of sim_create on a small
// grid.)  Whatever writes the word must have finished then; none (no word) is a no-op.
struct HostFlag {
    int32_t* word = nullptr;
    hipEvent_t event = nullptr;
    int device = 0;
};
hipError_t host_flag(HostFlag* f);
void host_flag_free(const HostFlag& f);

// Several host arrays placed in one device block and uploaded by one copy: add() returns an
// array's offset in the block.
struct UploadBlock {
    std::vector<char> host;
    template <class T>
    size_t add(const T* data, size_t count) {
        const size_t at = (host.size() + 255) / 256 * 256;
        host.resize(at + count * sizeof(T));
        if (count) std::memcpy(host.data() + at, data, count * sizeof(T));
        return at;
    }
    template <class T>
    size_t add(const std::vector<T>& v) {
        return add(v.data(), v.size());
    }
    hipError_t upload(char** block) const {
        *block = nullptr;
        const size_t bytes = host.empty() ? 1 : host.size();
        hipError_t e = device_malloc((void**)block, bytes);
        if (e == hipSuccess && !host.empty())
            e = hipMemcpy(*block, host.data(), host.size(), hipMemcpyHostToDevice);
        return e;
    }
};

}  // namespace cuesim
