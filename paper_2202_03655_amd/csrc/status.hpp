// Shared by the C ABI translation units: the reason of the last failure, kept
// per thread and returned by hdf_last_error(), and the product-timing switch.
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/hdf.h"

namespace hdf {
hdf_status set_error(hdf_status s, const std::string& msg);
void clear_error();
// Whether this thread's last failure was for want of device memory: the same call may succeed when less
// runs beside it.
bool failed_for_memory();
// Switch the HIP events around a factor's products on or off (hdf_info then
// reports no kernel times for them).  Products on many small factors use off.
void set_product_timing(hdf_handle h, bool on);
// Waits for everything enqueued on device `dev`, whichever device is current.
hipError_t wait_device(int dev);
// The library's caching device allocator: a block of at least b bytes, its size and device; a block is
// given back only when no enqueued work can use it.
// device_alloc is hipMalloc on the current device, tried again without the cache where memory is short.
hipError_t device_alloc(void** p, size_t b);
hipError_t pool_alloc(void** p, size_t b, size_t* got, int* dev);
void pool_release(void* p, size_t bytes, int dev);
// Products of several stored binary64 factors with one right-hand side each: the entries
// [pos, pos + n) of v and out belong to the factor at pos.  The factors outlive the batch.
struct ProductBatch;
hdf_status batch_create(const std::vector<hdf_handle>& factors, const std::vector<int64_t>& pos, hipStream_t s,
                        ProductBatch** out);
hdf_status batch_run(const ProductBatch* b, const double* v, double* out, hipStream_t s);
void batch_free(ProductBatch* b);
}  // namespace hdf
