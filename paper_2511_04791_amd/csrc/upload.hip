// Work lists from pinned host memory into the workspace.
//
// A kernel reads the staging buffer over the bus instead of a copy command: it queues like any
// launch, so the kernels behind it start at once, where a copy and the event that guards its buffer
// left the queue empty for about 6 us per call (4 requests' decode: 8 us from the copy's start to the
// first kernel, 3 us now; 690 KB of lists: 34 us, 18.5 us now).  The head of the workspace
// (error word, counters) is cleared here and not sent.
//
// Workgroup b reports that it has read its part by writing `seq` to flags[b] in host memory: the host
// may then reuse the buffer.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace duet {
namespace {

__global__ __launch_bounds__(256) void upload(const uint4* src, uint4* dst, int zero16, int n16, uint32_t* flags,
                                              uint32_t seq) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n16; i += gridDim.x * 256)
    dst[i] = i < zero16 ? make_uint4(0, 0, 0, 0) : src[i];
  __syncthreads();  // every wave has stored, and so has read, its part
  if (threadIdx.x == 0) __hip_atomic_store(flags + blockIdx.x, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

int upload_blocks(size_t bytes) { return (int)std::max<size_t>(1, std::min<size_t>(kUploadBlocks, bytes / 4096)); }

hipError_t launch_upload(const void* src, void* dst, size_t zero_bytes, size_t bytes, uint32_t* flags, uint32_t seq,
                         hipStream_t s) {
  hipLaunchKernelGGL(upload, dim3(upload_blocks(bytes)), dim3(256), 0, s, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), (int)(zero_bytes / 16), (int)(bytes / 16), flags, seq);
  return hipGetLastError();
}

}  // namespace duet
