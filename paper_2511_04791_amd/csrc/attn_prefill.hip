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
// unnormalised O^T) and stores it.  Of few pieces the last to finish combines the stored states in
// piece order, m = max(m_a, m_b), O = 2^(m_a - m) O_a + 2^(m_b - m) O_b (likewise the
// denominator), and writes the normalised rows; of more a merge kernel does.  Inside a piece a row may see no key at all
// (its position lies before the piece's first key): its state stays (-inf, 0, 0).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "attn_prefill_device.h"
#include "kernels.h"

namespace duet {
namespace {

using namespace prefill;

template <int D, int NH, bool kLean>
__global__ __launch_bounds__(kThreads, kLean ? 4 : 1) void prefill_bf16(AttnArgs a, WorkArgs w) {
  extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
  prefill_unit<D, NH, kLean>(a, w, blockIdx.x, lds);
}

// Heads of 64 hold half the ring and half the state of heads of 128, and their step is bound by the
// softmax's vector instructions and its dependency stalls, not by the matrix cores: two lean workgroups
// on a CU fill each other's stalls.  A lone lean workgroup is slower than a wide one, and with barely two
// items per CU all start at once, so that nothing evens out a CU that got two long ones.  Hence lean
// where every CU of the share gets two items and its mean load is at least 5/4 of the longest one.  Us a
// layer, wide against lean (16 / 2 heads):
//   512 items, load 1.5 / 2.0 / 3.0 times the longest (8192 tokens after 8192, 256 / 192 / 128 CUs)
//     524 / 698 / 1005 against 468 / 539 / 790;
//   280 items, load 1.27 (2048 tokens, 128 CUs) 49.7 against 43.3; on 192 and 256 CUs 40.6 and 31.3
//     against 38.1 and 31.5, but 292 items (2048 after 2048) on 256 CUs 59.7 against 64.8;
//   1280 items, load 1.0 (8192 tokens, 256 CUs) 184 against 197.
template <int D>
bool use_lean(const WorkArgs& w) {
  return D == 64 && w.n_pitems >= 2 * w.prefill_cus &&
         4 * w.prefill_tiles >= 5LL * w.prefill_longest * w.prefill_cus &&
         2 * PrefillSmem<D>::bytes(w.prefill_id_cap) <= kLdsBytes;
}

// Merges the pieces of every unit of more than kPrefillSelfMerge: one wave per (unit, wave of the unit,
// 32 dims), four pieces in flight, against the common max, sums in piece order.
template <int D, int NH>
__global__ __launch_bounds__(256) void prefill_merge(AttnArgs a, WorkArgs w) {
  constexpr int NO = D / 32;
  constexpr int WPH = kWaves / NH;
  const int lane = threadIdx.x & 63, hh = lane >> 5;
  const int job = 4 * blockIdx.x + uniform(threadIdx.x >> 6);
  const int unit = job / (kWaves * NO), wave = job / NO % kWaves, n = job % NO;
  if (unit >= w.n_punits) return;
  const PrefillUnit u = w.punits[unit];
  const int wrow0 = u.row0 + 32 * (wave % WPH);
  if (wrow0 >= u.q_len) return;
  const float2* const slot = reinterpret_cast<const float2*>(w.ppart) + (size_t)u.slot * kSlotPairs<D>;
  const float2* const o = slot + (size_t)(wave * NO + n) * 8 * 64 + lane;
  const float2* const ml = slot + (size_t)kThreads * (D / 4) + (size_t)wave * 64 + lane;
  float m = -INFINITY;
#pragma unroll 8
  for (int p = 0; p < u.pieces; ++p) m = fmaxf(m, ml[p * kSlotPairs<D>].x);
  float den = 0.f, num[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) num[v] = 0.f;
  for (int p0 = 0; p0 < u.pieces; p0 += 4) {
    float2 s[4], x[4][8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // pieces past the last re-read it
      const size_t at = (size_t)min(p0 + k, u.pieces - 1) * kSlotPairs<D>;
      s[k] = ml[at];
#pragma unroll
      for (int v2 = 0; v2 < 8; ++v2) x[k][v2] = o[at + v2 * 64];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (p0 + k >= u.pieces) break;
      // A piece whose keys all lie past a row's position holds (-inf, 0, 0) for it: weight 0.
      const float wgt = fast_exp2(s[k].x - m);
      den += wgt * s[k].y;
#pragma unroll
      for (int v2 = 0; v2 < 8; ++v2) {
        num[2 * v2] += wgt * x[k][v2].x;
        num[2 * v2 + 1] += wgt * x[k][v2].y;
      }
    }
  }
  const float inv = 1.0f / pair_sum(den);
  const int qi = wrow0 + (lane & 31);
  if (qi >= u.q_len) return;
  __bf16* op = reinterpret_cast<__bf16*>(a.out) + ((size_t)(u.q_start + qi) * a.h_q + u.head + wave / WPH) * D + 32 * n + 4 * hh;
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    __bf16 o4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o4[e] = static_cast<__bf16>(num[4 * g4 + e] * inv);
    *reinterpret_cast<uint2*>(op + 8 * g4) = __builtin_bit_cast(uint2, o4);
  }
}

template <int D, int NH>
hipError_t launch_merge(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  const int jobs = w.n_punits * kWaves * (D / 32);
  hipLaunchKernelGGL((prefill_merge<D, NH>), dim3((jobs + 3) / 4), dim3(256), 0, s, a, w);
  return hipGetLastError();
}

template <int D>
hipError_t launch_merge_nh(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  switch (prefill_heads_per_unit(a.group)) {
    case 1: return launch_merge<D, 1>(a, w, s);
    case 2: return launch_merge<D, 2>(a, w, s);
    case 4: return launch_merge<D, 4>(a, w, s);
    default: return launch_merge<D, 8>(a, w, s);
  }
}

template <int D, int NH, bool kLean>
hipError_t launch_bf16(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  if constexpr (D == 64 && !kLean) {
    if (use_lean<D>(w)) return launch_bf16<D, NH, true>(a, w, s);
  }
  static bool attr_set = false;  // the attribute is per function and process
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prefill_bf16<D, NH, kLean>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)PrefillSmem<D>::kMaxBytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((prefill_bf16<D, NH, kLean>), dim3(w.n_pitems), dim3(kThreads), PrefillSmem<D>::bytes(w.prefill_id_cap),
                     s, a, w);
  return hipGetLastError();
}

template <int D>
hipError_t launch_bf16_nh(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  switch (prefill_heads_per_unit(a.group)) {
    case 1: return launch_bf16<D, 1, false>(a, w, s);
    case 2: return launch_bf16<D, 2, false>(a, w, s);
    case 4: return launch_bf16<D, 4, false>(a, w, s);
    default: return launch_bf16<D, 8, false>(a, w, s);
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

size_t prefill_slot_bytes(int head_dim) {
  return (head_dim == 128 ? kSlotPairs<128> : kSlotPairs<64>) * sizeof(float2);
}

hipError_t launch_prefill(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  if (w.n_pitems == 0) return hipSuccess;
  if (a.dtype != 0) return launch_prefill_f32(a, w, s);
  const hipError_t e = a.head_dim == 128 ? launch_bf16_nh<128>(a, w, s) : launch_bf16_nh<64>(a, w, s);
  return e != hipSuccess ? e : launch_prefill_merge(a, w, s);
}

hipError_t launch_prefill_merge(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  if (w.n_punits == 0) return hipSuccess;
  return a.head_dim == 128 ? launch_merge_nh<128>(a, w, s) : launch_merge_nh<64>(a, w, s);
}

}  // namespace duet
