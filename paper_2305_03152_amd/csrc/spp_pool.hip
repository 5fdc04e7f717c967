// The library's device memory: what destroyed handles leave for the next ones.  Host code only.
#include "spp_pool.h"

#include <mutex>
#include <new>
#include <unordered_map>
#include <utility>
#include <vector>

namespace spp {

struct MemoryPool {
    std::mutex lock;
    std::vector<std::pair<void*, size_t>> kept;
    std::unordered_map<void*, size_t> lent;      // what pool_take has handed out
    size_t kept_bytes = 0;
    int contexts = 0;
    void trim() {
        for (auto& k : kept) (void)hipFree(k.first);
        kept.clear();
        kept_bytes = 0;
    }
};
static MemoryPool* pool_of(int device) {         // never destroyed: handles may outlive everything static
    static MemoryPool* pools = new (std::nothrow) MemoryPool[kPoolDevices];
    return pools && device >= 0 && device < kPoolDevices ? &pools[device] : nullptr;
}

hipError_t device_malloc(void** out, size_t bytes) {
    hipError_t e = hipMalloc(out, bytes);
    int device = 0;
    if (e != hipErrorOutOfMemory || hipGetDevice(&device) != hipSuccess) return e;
    pool_trim(device);
    (void)hipGetLastError();
    return hipMalloc(out, bytes);        // also where there was nothing to give: another thread may just have emptied the pool
}

hipError_t pool_take(int device, void** out, size_t bytes) {
    *out = nullptr;
    MemoryPool* p = pool_of(device);
    if (p) {
        std::lock_guard<std::mutex> hold(p->lock);
        size_t best = p->kept.size();
        for (size_t i = 0; i < p->kept.size(); ++i) {
            const size_t have = p->kept[i].second;
            if (have >= bytes && have <= bytes + bytes / 4 + 65536 && (best == p->kept.size() || have < p->kept[best].second)) best = i;
        }
        if (best < p->kept.size()) {
            const auto block = p->kept[best];
            try { p->lent[block.first] = block.second; } catch (...) { return hipErrorOutOfMemory; }
            p->kept[best] = p->kept.back();
            p->kept.pop_back();
            p->kept_bytes -= block.second;
            *out = block.first;
            return hipSuccess;
        }
    }
    const hipError_t e = device_malloc(out, bytes);
    if (e == hipSuccess && p) {
        std::lock_guard<std::mutex> hold(p->lock);
        try { p->lent[*out] = bytes; } catch (...) {}        // not known to the pool: freed when it is given back
    }
    return e;
}

static void give_back(int device, void* q, bool keep) {
    if (!q) return;
    MemoryPool* p = pool_of(device);
    if (p) {
        std::lock_guard<std::mutex> hold(p->lock);
        const auto it = p->lent.find(q);
        if (it != p->lent.end()) {
            const size_t bytes = it->second;
            p->lent.erase(it);
            if (keep && p->contexts > 0 && p->kept_bytes + bytes <= kPoolBytes) {
                try {
                    p->kept.emplace_back(q, bytes);
                    p->kept_bytes += bytes;
                    return;
                } catch (...) {}
            }
        }
    }
    (void)hipFree(q);
}

void pool_give(int device, void* q) { give_back(device, q, true); }

void pool_retire(int device, std::initializer_list<void*> blocks) {
    // A wait that is refused (another thread may be capturing a graph) leaves work in flight that the next owner's would meet:
    // such memory goes to hipFree, which does not hand it on before that work has ended.
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    for (void* q : blocks) give_back(device, q, idle);
}

void pool_trim(int device) {
    MemoryPool* p = pool_of(device);
    if (!p) return;
    std::lock_guard<std::mutex> hold(p->lock);
    p->trim();
}

void pool_context(int device, int change) {
    MemoryPool* p = pool_of(device);
    if (!p) return;
    std::lock_guard<std::mutex> hold(p->lock);
    p->contexts += change;
    if (p->contexts == 0) p->trim();
}

}  // namespace spp
