// Decode attention over the paged KV cache: split-K partial kernel and reduce kernel.
//
// Each decode request has one query token at absolute position kv_len - 1 that attends all
// kv_len keys (paper, Section 2: the new token's key and value are appended before attention;
// Section 4.1: decode is q = 1, c > 0).  The work is HBM-bound: every key and value is read
// once.  A work item is (request, kv head, split) where a split is a run of logical pages of a
// length that the batch fixes (kernels.h, decode_rule).  One wave owns one item and reads each page
// of its kv head once for all query heads of the GQA group, so the bytes moved are the algorithmic
// K/V bytes.
//
// bf16 path, per page (16 tokens), on MFMA with fp32 accumulate:
//   S^T [16 tokens x 16 heads] = K_page [16 x d] . Q^T [d x 16]   (16x16x32, one per 32 dims)
//   O^T [16 dims x 16 heads]  += V^T   [16 x 16] . P^T [16 x 16]  (16x16x16, one per 16 dims)
// Heads beyond the group size are zero columns.  K is read token-major (16 B per lane, the
// MFMA A layout); V pages are stored dim-major, so a lane's 4 consecutive tokens of one dim
// are 8 contiguous bytes and P^T never leaves registers.  Pages cycle through four register
// buffers, so three pages are in flight while one is computed, across item boundaries too.
// Online softmax keeps a reference max per head that only moves when a score exceeds it by
// more than 2^8 (base-2 units), so the output rescale is rare.  Partials (unnormalised output,
// reference max, denominator) go to the workspace, and one wave per (request, query head) merges
// the splits: the reduce kernel, or, for the layers of a call but the last, the next layer's bf16
// partial kernel, in the waves whose item queue has run dry.
//
// A batch of few items (kernels.h, decode_rule) cannot fill the chip with one wave per item: it runs
// one workgroup per item instead (decode_small_bf16).
// All arithmetic order depends on logical token positions only.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "attn_decode_device.h"
#include "kernels.h"
#include "wave_ops.h"

namespace duet {
namespace {

using namespace decode;

template <int D, int PPS>
__global__ __launch_bounds__(256, 1) void decode_partial_bf16(AttnArgs a, WorkArgs w) {
  __shared__ __align__(16) float stage[4][kStageFloats];
  if (blockIdx.x == 0) clear_previous_counters(w);
  const int wave = uniform(threadIdx.x >> 6);
  decode_stream<D, PPS>(a, w, stage[wave], 4 * blockIdx.x + wave, 4 * gridDim.x);
}

template <int D, bool kPack>
__global__ __launch_bounds__(kSmallThreads, 4) void decode_small_bf16(AttnArgs a, WorkArgs w) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  decode_items<D, kPack>(a, w, blockIdx.x, lds);
}

// Merges every (decode request, query head) pair of one layer: one wave per pair.
template <int D, typename OutT>
__global__ __launch_bounds__(256) void decode_reduce(AttnArgs a, WorkArgs w) {
  // The partial kernel before this one on the stream has finished with its counter set: clear it
  // for the next call.
  if (blockIdx.x == 0 && threadIdx.x < kDecodeSetLines) w.work_counter[threadIdx.x * kDecodeQueueStride] = 0;
  const int pair = blockIdx.x * 4 + uniform(threadIdx.x >> 6);
  if (pair >= w.n_dreq * a.h_q) return;
  merge_pair<D, OutT>(a, w, w.pacc, w.pml, a.out, pair, threadIdx.x & 63);
}

}  // namespace

constexpr int kMinRounds = 4;      // items per wave the persistent grid is sized for, at least
constexpr int kMinWavesPerCu = 4;  // waves per CU of the share, at least

// Persistent grid size.  The memory system needs far fewer waves in flight than fit, so the grid
// is sized for at least kMinRounds items per wave (a short tail when the last items
// finish), but never below kMinWavesPerCu waves per CU (bandwidth on small CU
// shares) nor above what is resident at once.
template <int D, int PPS>
hipError_t launch_persistent(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  static int per_cu = 0;  // resident 256-thread blocks per CU, from the occupancy calculator
  if (per_cu == 0) {
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void*>(&decode_partial_bf16<D, PPS>), 256, 0);
    if (e != hipSuccess) return e;
    if (per_cu < 1) per_cu = 1;
  }
  const int capacity = w.decode_cus * per_cu * 4;
  const int floor_waves = w.decode_cus * kMinWavesPerCu;
  const int want = (w.n_ditems + kMinRounds - 1) / kMinRounds;
  const int waves = std::max(1, std::min(capacity, std::max(want, floor_waves)));
  hipLaunchKernelGGL((decode_partial_bf16<D, PPS>), dim3((waves + 3) / 4), dim3(256), 0, s, a, w);
  return hipGetLastError();
}

template <int D, bool kPack>
hipError_t launch_small(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  static bool attr_set = false;  // the attribute is per function and process
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_small_bf16<D, kPack>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)small_lds_bytes<D>(16));
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((decode_small_bf16<D, kPack>), dim3(small_blocks(w)), dim3(kSmallThreads), small_lds_bytes<D>(a.group), s, a, w);
  return hipGetLastError();
}

hipError_t launch_decode_partial(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  if (w.n_dreq == 0) return hipSuccess;
  if (a.dtype != 0) return launch_decode_partial_f32(a, w, s);
  if (w.decode_small && w.n_small8 < w.n_ditems)
    return a.head_dim == 128 ? launch_small<128, true>(a, w, s) : launch_small<64, true>(a, w, s);
  if (w.decode_small) return a.head_dim == 128 ? launch_small<128, false>(a, w, s) : launch_small<64, false>(a, w, s);
  if (w.decode_pps == kDecodePagesPerSplitShort)
    return a.head_dim == 128 ? launch_persistent<128, kDecodePagesPerSplitShort>(a, w, s)
                             : launch_persistent<64, kDecodePagesPerSplitShort>(a, w, s);
  return a.head_dim == 128 ? launch_persistent<128, kDecodePagesPerSplit>(a, w, s)
                           : launch_persistent<64, kDecodePagesPerSplit>(a, w, s);
}

hipError_t launch_decode_reduce(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  if (w.n_dreq == 0 || (w.decode_small && w.max_split == 1)) return hipSuccess;  // nothing to merge
  const dim3 grid((w.n_dreq * a.h_q + 3) / 4);
  if (a.dtype == 0) {
    if (a.head_dim == 128) hipLaunchKernelGGL((decode_reduce<128, __bf16>), grid, dim3(256), 0, s, a, w);
    else hipLaunchKernelGGL((decode_reduce<64, __bf16>), grid, dim3(256), 0, s, a, w);
  } else {
    if (a.head_dim == 128) hipLaunchKernelGGL((decode_reduce<128, float>), grid, dim3(256), 0, s, a, w);
    else hipLaunchKernelGGL((decode_reduce<64, float>), grid, dim3(256), 0, s, a, w);
  }
  return hipGetLastError();
}

}  // namespace duet
