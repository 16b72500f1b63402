// Buffer resources: loads and stores of byte offsets that are checked against the tensor's extent.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace distdl {

constexpr uint32_t kOob = 0x7ffffff0u;  // an offset that fails the range check of every buffer (tensors are < 2 GiB)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

}  // namespace distdl
