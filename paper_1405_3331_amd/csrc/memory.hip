// memory.hip -- reuse of device memory between the library's objects (host code).
//
// A parameter fit creates and destroys a simulation per iteration and a gradient replaces its
// record per run: the same sizes again and again.  From the runtime that costs about 40
// allocations and as many frees per iteration (600 us, each free waiting for the device), and
// memory given back to the driver is cleared before it can be had again (34 GB/s, 250 ms for the
// 8.4 GB of field states of 2000 steps at 1024^2).
//
// Idle blocks are bounded: a sixteenth of a device's memory while any object is alive, kIdleRest
// between objects, the longest idle given back first; all of a device's are given back when an
// allocation fails, and all of them by release_device_memory.
#include <algorithm>
#include <list>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>

#include "memory.hpp"

namespace cuesim {

namespace {

constexpr size_t kBusyShare = 16;
constexpr size_t kIdleRest = (size_t)1 << 30;

struct Block {
    void* p;
    size_t bytes;
    int device;
};

struct Device {
    size_t idle = 0;   // bytes
    size_t busy = 0;   // idle bytes to keep while an object lives (0: not asked for yet)
    std::vector<HostFlag> flags;   // idle ones
};

struct Pool {
    std::mutex lock;
    std::unordered_map<void*, Block> live;
    std::list<Block> idle;   // longest idle first
    std::multimap<std::pair<int, size_t>, std::list<Block>::iterator> by_size;
    std::map<int, Device> devices;
    int users = 0;
    std::vector<int32_t*> words;   // pinned ones of no flag yet

    void forget(std::list<Block>::iterator b) {
        auto r = by_size.equal_range({b->device, b->bytes});
        for (auto k = r.first; k != r.second; ++k)
            if (k->second == b) {
                by_size.erase(k);
                break;
            }
        devices[b->device].idle -= b->bytes;
        idle.erase(b);
    }
    // Idle bytes to keep on a device as things are.
    size_t limit(int device) {
        Device& d = devices[device];
        if (d.busy == 0) {
            size_t total = 0;
            if (hipDeviceTotalMem(&total, device) != hipSuccess) {
                (void)hipGetLastError();
                total = 0;
            }
            d.busy = std::max<size_t>(total / kBusyShare, 1);
        }
        return users > 0 ? d.busy : std::min(d.busy, kIdleRest);
    }
    // Blocks to give back so that no device (`device` only, if >= 0) keeps more than its limit,
    // or any idle block at all.
    std::vector<Block> trim(bool all, int device = -1) {
        std::vector<Block> out;
        for (auto b = idle.begin(); b != idle.end();) {
            const auto next = std::next(b);
            if ((device < 0 || b->device == device) &&
                (all || devices[b->device].idle > limit(b->device))) {
                out.push_back(*b);
                forget(b);
            }
            b = next;
        }
        return out;
    }
};

// never destroyed: objects may be released while the process ends
Pool& pool() {
    static Pool* p = new Pool;
    return *p;
}

hipError_t give_back(const std::vector<Block>& blocks) {
    hipError_t e = hipSuccess;
    for (const Block& b : blocks) {
        const hipError_t f = hipFree(b.p);
        if (f != hipSuccess) e = f;
    }
    return e;
}

size_t rounded(size_t bytes) {
    const size_t unit = bytes < ((size_t)1 << 20) ? 512 : (size_t)64 << 10;
    return (std::max<size_t>(bytes, 1) + unit - 1) / unit * unit;
}

}  // namespace

hipError_t device_malloc(void** p, size_t bytes) {
    *p = nullptr;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    const size_t need = rounded(bytes);
    Pool& q = pool();
    {
        std::lock_guard<std::mutex> hold(q.lock);
        const auto k = q.by_size.lower_bound({device, need});
        if (k != q.by_size.end() && k->first.first == device && k->first.second <= need + need / 4) {
            const Block b = *k->second;
            q.forget(k->second);
            q.live.emplace(b.p, b);
            *p = b.p;
            return hipSuccess;
        }
    }
    e = hipMalloc(p, need);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        std::vector<Block> out;
        {
            std::lock_guard<std::mutex> hold(q.lock);
            out = q.trim(true, device);
        }
        if (out.empty()) return e;
        (void)give_back(out);
        e = hipMalloc(p, need);
        if (e != hipSuccess) return e;
    }
    std::lock_guard<std::mutex> hold(q.lock);
    q.live.emplace(*p, Block{*p, need, device});
    return hipSuccess;
}

void device_free(void* p) {
    if (!p) return;
    Pool& q = pool();
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> hold(q.lock);
        const auto k = q.live.find(p);
        if (k == q.live.end()) return;
        q.idle.push_back(k->second);
        q.live.erase(k);
        const auto b = std::prev(q.idle.end());
        q.by_size.emplace(std::make_pair(b->device, b->bytes), b);
        q.devices[b->device].idle += b->bytes;
        if (q.devices[b->device].idle > q.limit(b->device)) out = q.trim(false, b->device);
    }
    (void)give_back(out);
}

hipError_t release_device_memory() {
    Pool& q = pool();
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> hold(q.lock);
        out = q.trim(true);
    }
    return give_back(out);
}

hipError_t host_flag(HostFlag* f) {
    constexpr size_t kLine = 64, kPage = 4096;
    *f = HostFlag{};
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    Pool& q = pool();
    std::lock_guard<std::mutex> hold(q.lock);
    std::vector<HostFlag>& idle = q.devices[device].flags;
    if (idle.empty()) {
        if (q.words.empty()) {
            char* page = nullptr;
            e = hipHostMalloc((void**)&page, kPage, hipHostMallocPortable);
            if (e != hipSuccess) return e;
            for (size_t at = 0; at < kPage; at += kLine) q.words.push_back((int32_t*)(page + at));
        }
        HostFlag n;
        e = hipEventCreateWithFlags(&n.event, hipEventDisableTiming);
        if (e != hipSuccess) return e;
        n.word = q.words.back();
        n.device = device;
        q.words.pop_back();
        idle.push_back(n);
    }
    *f = idle.back();
    idle.pop_back();
    *f->word = 0;
    return hipSuccess;
}

void host_flag_free(const HostFlag& f) {
    if (!f.word) return;
    Pool& q = pool();
    std::lock_guard<std::mutex> hold(q.lock);
    q.devices[f.device].flags.push_back(f);
}

size_t device_idle_bytes(int device) {
    Pool& q = pool();
    std::lock_guard<std::mutex> hold(q.lock);
    return q.devices[device].idle;
}

void device_memory_user(int change) {
    Pool& q = pool();
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> hold(q.lock);
        q.users += change;
        if (q.users == 0)
            for (const auto& d : q.devices)
                if (d.second.idle > q.limit(d.first))
                    for (const Block& b : q.trim(false, d.first)) out.push_back(b);
    }
    (void)give_back(out);
}

}  // namespace cuesim
