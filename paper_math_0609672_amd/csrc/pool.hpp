#pragma once

#include <hip/hip_runtime_api.h>

#include <cstddef>

namespace srw {

// Device memory from the library's kept blocks (pool.cpp).  dev_release: no work on the
// block may be pending (the caller has synchronised); it may be called from any thread.
// dev_trim gives every kept block back to the device.
hipError_t dev_alloc(void** out, size_t bytes);
void dev_release(void* p);
void dev_trim(int dev);

// hipMallocAsync on s, for calls that do not synchronise; where memory is short, once more
// without the kept blocks.
hipError_t stream_alloc(void** out, size_t bytes, hipStream_t s);

}  // namespace srw
