// Device memory.  The pool keeps what destroyed graphs and caches held, at most kPoolBytes per device, for the next ones (a graph
// of 121M edges: 484 MB, which the driver maps and clears again at every allocation, 0.1 to 100 ms); it is given back with the
// device's last context, on request, and to any allocation of the library that would fail without it: all of them go through
// device_malloc, which is hipMalloc that then empties the pool and tries again.  Allocations of the program outside the library
// cannot do that; spp_memory_trim is for them.  Safe with several threads.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>

#include <initializer_list>

namespace spp {

constexpr size_t kPoolBytes = (size_t)1 << 30;
constexpr int kPoolDevices = 64;                 // devices beyond have no pool
hipError_t device_malloc(void** out, size_t bytes);
hipError_t pool_take(int device, void** out, size_t bytes);
void pool_give(int device, void* p);             // memory that no stream uses any more, on the current device
void pool_retire(int device, std::initializer_list<void*> blocks);       // waits for the current device, then gives them back
void pool_trim(int device);                      // gives back what is kept
void pool_context(int device, int change);       // contexts of the device: +1, -1
template <class T> hipError_t device_malloc(T** out, size_t bytes) { return device_malloc(reinterpret_cast<void**>(out), bytes); }
template <class T> hipError_t pool_take(int device, T** out, size_t bytes) { return pool_take(device, reinterpret_cast<void**>(out), bytes); }

}  // namespace spp
