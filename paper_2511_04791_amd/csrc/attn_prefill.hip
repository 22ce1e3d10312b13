// Prefill-chunk attention over the paged KV cache (causal, with a cached prefix).
//
// A prefill request schedules q tokens after c cached ones; its keys and values, including
// those of the q new tokens, are already in the cache (paper, Section 2).  Query i sits at
// absolute position c + i and attends keys 0 .. c + i (Section 4.1: chunked prefill is q > 1,
// c > 0).  The work is a dense contraction, so it runs on MFMA: bf16 operands, fp32 accumulate.
//
// Work unit: one workgroup of 8 waves owns NH query heads of one GQA group (NH = group size, at
// most 8) and 256 / NH consecutive queries; each wave owns 32 (head, query) rows.  All waves of
// the unit read the same keys, so each K/V tile is fetched once for NH heads.  Keys stream
// through LDS 64 at a time (4 pages) in a 4-slot ring: K as [64 keys][d] and V as
// V^T [d][64 keys] (V pages are stored dim-major, so staging V^T is a straight copy).  Per
// 64-key step each wave computes, on the 32x32x16 bf16 MFMA,
//   S^T [64 keys x 32 queries] = K . Q^T       (Q^T held in registers for the whole loop)
//   O^T [d x 32 queries]      += V^T . P^T     (P^T never leaves registers)
// With S^T and O^T transposed, every per-query quantity (running max, denominator, rescale
// factor) lives in one lane pair (lane, lane ^ 32), so the online softmax needs one cross-lane
// exchange per step.  Rows of the K tile are fed to the MFMA in an order that makes each
// lane's score registers hold 8 consecutive keys, exactly the B layout P^T needs.
// The running max is only moved when a score exceeds it by more than 2^8 (in base-2 units);
// otherwise probabilities are taken against the stale max.  The result is the same softmax
// (numerator and denominator share the reference), and the O rescale is skipped on most steps.
// Key tiles past a wave's last query are skipped; only tiles crossing the diagonal are masked.
//
// A unit with a long key range may run as several pieces, each over a run of its key tiles
// (kernels.h).  A piece keeps the same per-row state as a whole unit (reference max, denominator,
// unnormalised O^T) and stores it; the last piece of the unit to finish combines the stored
// states in piece order, m = max(m_a, m_b), O = 2^(m_a - m) O_a + 2^(m_b - m) O_b (likewise the
// denominator), and writes the normalised rows.  Inside a piece a row may see no key at all
// (its position lies before the piece's first key): its state stays (-inf, 0, 0).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "attn_prefill_device.h"
#include "kernels.h"

namespace duet {
namespace {

using namespace prefill;

template <int D, int NH>
__global__ __launch_bounds__(kThreads, 1) void prefill_bf16(AttnArgs a, WorkArgs w) {
  extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
  prefill_unit<D, NH>(a, w, blockIdx.x, lds);
}

template <int D, int NH>
hipError_t launch_bf16(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  static bool attr_set = false;  // the attribute is per function and process
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prefill_bf16<D, NH>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)PrefillSmem<D>::kMaxBytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((prefill_bf16<D, NH>), dim3(w.n_pitems), dim3(kThreads), PrefillSmem<D>::bytes(w.prefill_id_cap),
                     s, a, w);
  return hipGetLastError();
}

template <int D>
hipError_t launch_bf16_nh(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  switch (prefill_heads_per_unit(a.group)) {
    case 1: return launch_bf16<D, 1>(a, w, s);
    case 2: return launch_bf16<D, 2>(a, w, s);
    case 4: return launch_bf16<D, 4>(a, w, s);
    default: return launch_bf16<D, 8>(a, w, s);
  }
}

}  // namespace

int prefill_heads_per_unit(int group) {
  // largest power of two <= min(group, waves per workgroup) that divides the group
  int nh = 1;
  while (nh * 2 <= kWaves && group % (nh * 2) == 0) nh *= 2;
  return nh;
}

int prefill_rows_per_unit(int group, int dtype) {
  return dtype == 0 ? 32 * kWaves / prefill_heads_per_unit(group) : kPrefillRows;
}

int prefill_piece_tiles_for(long long total_tiles) {
  const long long even = (total_tiles + kPrefillPieceFill - 1) / kPrefillPieceFill;
  return (int)std::max<long long>(kPrefillPieceMinTiles, even);
}

size_t prefill_slot_bytes(int head_dim) { return (size_t)kThreads * (head_dim / 2 + 2) * sizeof(float); }

hipError_t launch_prefill(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  if (w.n_pitems == 0) return hipSuccess;
  if (a.dtype == 0) return a.head_dim == 128 ? launch_bf16_nh<128>(a, w, s) : launch_bf16_nh<64>(a, w, s);
  return launch_prefill_f32(a, w, s);
}

}  // namespace duet
