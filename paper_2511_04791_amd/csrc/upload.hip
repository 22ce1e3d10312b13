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
//
// A graph that captured an upload reads its source again at every replay, long after the buffer has
// gone to other calls.  Under capture the lists therefore travel inside the graph, as kernel
// arguments of 3.5 KB each (most lists are a few KB).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

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

constexpr int kChunkWords = 896;
struct Chunk {
  uint32_t w[kChunkWords];
};
__global__ __launch_bounds__(256) void store_chunk(Chunk c, uint32_t* dst, int n) {
  for (int i = threadIdx.x; i < n; i += 256) dst[i] = c.w[i];
}

}  // namespace

int upload_blocks(size_t bytes) { return (int)std::max<size_t>(1, std::min<size_t>(kUploadBlocks, bytes / 4096)); }

hipError_t launch_upload(const void* src, void* dst, size_t zero_bytes, size_t bytes, uint32_t* flags, uint32_t seq,
                         hipStream_t s) {
  hipLaunchKernelGGL(upload, dim3(upload_blocks(bytes)), dim3(256), 0, s, static_cast<const uint4*>(src),
                     static_cast<uint4*>(dst), (int)(zero_bytes / 16), (int)(bytes / 16), flags, seq);
  return hipGetLastError();
}

hipError_t launch_upload_by_value(const void* src, void* dst, size_t bytes, hipStream_t s) {
  for (size_t at = 0; at < bytes; at += sizeof(Chunk)) {
    Chunk c;
    const size_t n = std::min(sizeof(Chunk), bytes - at);
    std::memcpy(c.w, static_cast<const char*>(src) + at, n);
    hipLaunchKernelGGL(store_chunk, dim3(1), dim3(256), 0, s, c, reinterpret_cast<uint32_t*>(static_cast<char*>(dst) + at),
                       (int)(n / 4));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace duet
