// Both halves of one aggregated bf16 layer in one launch.
//
// Decode streams keys and values and leaves the matrix cores idle; prefill keeps them busy and hardly
// reads.  One after the other, each half leaves the other's resource unused, and each ends with a tail
// of its own.  Here the first `decode_blocks` workgroups are decode's persistent waves, the next ones
// the prefill items, longest first, and the last ones more decode waves, which join the item queues as
// CUs run out of prefill work: whichever half lasts longer ends on every CU.
//
// With heads of 128 a workgroup of either kind fills a CU (the prefill ring takes its LDS).  With heads of
// 64 the ring is 64 of 160 KiB and registers are the limit: eight waves of 156 leave no room for eight
// more, but a decode workgroup, four of whose waves end at once, does.  While prefill items last,
// decode runs on decode_blocks CUs: the number at which four waves each keep the memory busy (a wave
// streams about 10 GB/s; eight waves per CU halve that and leave each twice as long with its
// last item).  One layer of 64 decodes (452 MB) beside 2048 new tokens, Llama-3-8B: decode 92 us and
// prefill 52 us apart; together 139 / 126 / 122 / 130 us with 96 / 128 / 160 / 192 decode blocks of
// four waves, and 134 us with 160 blocks of eight.  Heads of 64 read half as much per page and want
// more (100 decodes beside 2048 tokens: 65 / 64 / 57 us with 128 / 160 / 192 blocks).
//
// A batch of few or short decode items (decode_small) runs them first, as launched alone.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "attn_decode_device.h"
#include "attn_prefill_device.h"
#include "kernels.h"

namespace duet {
namespace {

constexpr int kMixedWaves = 4;  // decode waves per workgroup
template <int D>
constexpr int kMixedDecodeBlocks = D == 128 ? 160 : 192;

// Streamed decode keeps its finished items in the prefill ring's LDS.
template <int D>
constexpr size_t kRingBytes = prefill::PrefillSmem<D>::kTileBytes;
static_assert(kMixedWaves * decode::kStageFloats * sizeof(float) <= kRingBytes<64>, "the waves' buffers fit");
static_assert(decode::small_lds_bytes<128>(16) <= kRingBytes<128> && decode::small_lds_bytes<64>(16) <= kRingBytes<64>,
              "a small item fits");
static_assert(decode::kSmallThreads == prefill::kThreads, "one workgroup size");

// PPS: pages of a streamed decode item; 0: small items, -1: of which some share a workgroup.
template <int D, int NH, int PPS>
__global__ __launch_bounds__(prefill::kThreads, 2) void mixed_bf16(AttnArgs a, WorkArgs w, int decode_blocks) {
  extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
  const int b = blockIdx.x;
  if (b >= decode_blocks && b < decode_blocks + w.n_pitems) {
    prefill::prefill_unit<D, NH, false>(a, w, b - decode_blocks, lds);
    return;
  }
  float* const fl = reinterpret_cast<float*>(lds);
  if constexpr (PPS <= 0) {
    decode::decode_items<D, PPS < 0>(a, w, b, fl);
  } else {
    if (b == 0) decode::clear_previous_counters(w);
    const int wave = uniform(threadIdx.x >> 6);
    if (wave >= kMixedWaves) return;
    const int block = b < decode_blocks ? b : b - w.n_pitems;
    decode::decode_stream<D, PPS>(a, w, fl + wave * decode::kStageFloats, kMixedWaves * block + wave,
                                  kMixedWaves * decode_blocks);
  }
}

template <int D, int NH, int PPS>
hipError_t launch(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  using Smem = prefill::PrefillSmem<D>;
  static bool attr_set = false;  // the attribute is per function and process
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&mixed_bf16<D, NH, PPS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)Smem::kMaxBytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  // Streamed: multiples of 8 (one per XCD), and at least two items for each of the first waves.
  const int first = PPS <= 0 ? small_blocks(w)
                             : std::max(8, std::min(kMixedDecodeBlocks<D>, w.n_ditems / (2 * kMixedWaves) / 8 * 8));
  const int late = PPS <= 0 ? 0 : std::max(0, w.decode_cus - first);
  hipLaunchKernelGGL((mixed_bf16<D, NH, PPS>), dim3(first + w.n_pitems + late), dim3(prefill::kThreads),
                     Smem::bytes(w.prefill_id_cap), s, a, w, first);
  return hipGetLastError();
}

template <int D, int NH>
hipError_t launch_pps(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  if (w.decode_small) return w.n_small8 < w.n_ditems ? launch<D, NH, -1>(a, w, s) : launch<D, NH, 0>(a, w, s);
  if (w.decode_pps == kDecodePagesPerSplitShort) return launch<D, NH, kDecodePagesPerSplitShort>(a, w, s);
  return launch<D, NH, kDecodePagesPerSplit>(a, w, s);
}

template <int D>
hipError_t launch_nh(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  switch (prefill_heads_per_unit(a.group)) {
    case 1: return launch_pps<D, 1>(a, w, s);
    case 2: return launch_pps<D, 2>(a, w, s);
    case 4: return launch_pps<D, 4>(a, w, s);
    default: return launch_pps<D, 8>(a, w, s);
  }
}

}  // namespace

hipError_t launch_mixed(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  const hipError_t e = a.head_dim == 128 ? launch_nh<128>(a, w, s) : launch_nh<64>(a, w, s);
  return e != hipSuccess ? e : launch_prefill_merge(a, w, s);
}

}  // namespace duet
