// Device memory.  device_malloc is hipMalloc that gives the pool's memory back and tries again before it fails.  The pool
// keeps what destroyed graphs and caches held, at most kPoolBytes per device, for the next ones (a graph of 121M edges: 484 MB,
// which the driver maps and clears again at every allocation, 0.1 to 100 ms); it is given back with the device's last context.
// Safe with several threads.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>

#include <initializer_list>

namespace spp {

constexpr size_t kPoolBytes = (size_t)1 << 30;
hipError_t device_malloc(void** out, size_t bytes);
hipError_t pool_take(int device, void** out, size_t bytes);
void pool_give(int device, void* p);             // memory that no stream uses any more, on the current device
void pool_retire(int device, std::initializer_list<void*> blocks);       // waits for the current device, then gives them back
void pool_context(int device, int change);       // contexts of the device: +1, -1
template <class T> hipError_t pool_take(int device, T** out, size_t bytes) { return pool_take(device, reinterpret_cast<void**>(out), bytes); }

}  // namespace spp
