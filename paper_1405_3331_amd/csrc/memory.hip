// memory.hip -- reuse of device memory between the library's objects (host code).
//
// A parameter fit creates and destroys a simulation per iteration and a gradient replaces its
// record per run: the same sizes again and again.  From the runtime that costs about 40
// allocations and as many frees per iteration (600 us, each free waiting for the device), and
// memory given back to the driver is cleared before it can be had again (34 GB/s): a loop of
// 2000-step gradients at 1024^2, with 10 GB of recorded states each, ran at 17 ms per pass
// until the cleared memory was used up and at 250 ms from then on.
//
// Idle blocks are bounded: kIdleBusy bytes while any object is alive, kIdleRest between
// objects, the longest idle given back first; and all of a device's are given back when an
// allocation fails.
#include <algorithm>
#include <list>
#include <map>
#include <mutex>
#include <unordered_map>

#include "memory.hpp"

namespace cuesim {

namespace {

constexpr size_t kIdleBusy = (size_t)12 << 30;   // of 288 GB; the record of that gradient is 10
constexpr size_t kIdleRest = (size_t)1 << 30;

struct Block {
    void* p;
    size_t bytes;
    int device;
};

struct Pool {
    std::mutex lock;
    std::unordered_map<void*, Block> live;
    std::list<Block> idle;   // longest idle first
    std::multimap<std::pair<int, size_t>, std::list<Block>::iterator> by_size;
    size_t idle_bytes = 0;
    int users = 0;
    std::vector<int32_t*> words;   // free pinned words

    void forget(std::list<Block>::iterator b) {
        auto r = by_size.equal_range({b->device, b->bytes});
        for (auto k = r.first; k != r.second; ++k)
            if (k->second == b) {
                by_size.erase(k);
                break;
            }
        idle_bytes -= b->bytes;
        idle.erase(b);
    }
    // Blocks to give back so that at most `limit` bytes stay (of `device` only, if >= 0).
    std::vector<Block> trim(size_t limit, int device = -1) {
        std::vector<Block> out;
        for (auto b = idle.begin(); b != idle.end() && idle_bytes > limit;) {
            const auto next = std::next(b);
            if (device < 0 || b->device == device) {
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

void give_back(const std::vector<Block>& blocks) {
    for (const Block& b : blocks) (void)hipFree(b.p);
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
            out = q.trim(0, device);
        }
        if (out.empty()) return e;
        give_back(out);
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
        q.idle_bytes += b->bytes;
        out = q.trim(q.users > 0 ? kIdleBusy : kIdleRest);
    }
    give_back(out);
}

hipError_t pinned_word(int32_t** p) {
    constexpr size_t kLine = 64, kPage = 4096;
    *p = nullptr;
    Pool& q = pool();
    std::lock_guard<std::mutex> hold(q.lock);
    if (q.words.empty()) {
        char* page = nullptr;
        const hipError_t e = hipHostMalloc((void**)&page, kPage, hipHostMallocPortable);
        if (e != hipSuccess) return e;
        for (size_t at = 0; at < kPage; at += kLine) q.words.push_back((int32_t*)(page + at));
    }
    *p = q.words.back();
    q.words.pop_back();
    **p = 0;
    return hipSuccess;
}

void pinned_word_free(int32_t* p) {
    if (!p) return;
    Pool& q = pool();
    std::lock_guard<std::mutex> hold(q.lock);
    q.words.push_back(p);
}

size_t device_idle_bytes(int device) {
    Pool& q = pool();
    std::lock_guard<std::mutex> hold(q.lock);
    size_t n = 0;
    for (const Block& b : q.idle) n += b.device == device ? b.bytes : 0;
    return n;
}

void device_memory_user(int change) {
    Pool& q = pool();
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> hold(q.lock);
        q.users += change;
        if (q.users == 0) out = q.trim(kIdleRest);
    }
    give_back(out);
}

}  // namespace cuesim
