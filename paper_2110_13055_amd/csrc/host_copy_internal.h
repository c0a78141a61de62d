// host_copy_internal.h -- large device-to-host copies (host_copy.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cdi {

// Copies from this size on go through the staging area.
constexpr uint64_t kStagedCopyMin = 16ull << 20;

// bytes from device memory to pageable host memory, ordered on s; the copy is
// complete on return. Any thread, any stream.
hipError_t copy_to_host(void *dst, const void *src, uint64_t bytes, hipStream_t s);

// The staging area lives while any solver does: one call when a solver is
// made, one when it is destroyed.
void staging_user_added();
void staging_user_removed();

}  // namespace cdi
