// Device helpers shared by the attention kernels (internal).
#pragma once

#include <hip/hip_runtime.h>

namespace duet {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ bool page_ok(int id, long long num_phys) { return id >= 0 && (long long)id < num_phys; }

// Combine a value across the four 16-lane rows of a wave (lanes l, l ^ 16, l ^ 32, l ^ 48) with
// the row-swap permutes, which stay in the vector ALU: an LDS permute would be counted with the
// scalar loads, so waiting for it would also wait for them.
__device__ __forceinline__ float max_rows(float x) {
  const unsigned u = __float_as_uint(x);
  auto s32 = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const float m = fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
  const unsigned v = __float_as_uint(m);
  auto s16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
}
__device__ __forceinline__ float sum_rows(float x) {
  const unsigned u = __float_as_uint(x);
  auto s16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float m = __uint_as_float(s16[0]) + __uint_as_float(s16[1]);  // rows (0+1, 0+1, 2+3, 2+3)
  const unsigned v = __float_as_uint(m);
  auto s32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __uint_as_float(s32[0]) + __uint_as_float(s32[1]);
}

// The last request r of [0, n) with before(r), where before(0) holds and before is true up to some
// request and false from there on.  A whole wave searches 64-ary: one memory round trip up to 64
// requests, two up to 4096.
template <typename F>
__device__ __forceinline__ int find_request(int n, F before) {
  const int lane = threadIdx.x & 63;
  int lo = 0, end = n;
  while (end - lo > 1) {
    const int step = (end - lo + 63) / 64;
    const int x = lo + lane * step;
    const int k = __popcll(__ballot(x < end && before(x)));
    lo += (max(k, 1) - 1) * step;
    end = min(end, lo + step);
  }
  return lo;
}

// The byte permutes that gather the low (high) halves of two words: (a.lo, b.lo), (a.hi, b.hi).
__device__ __forceinline__ unsigned lows(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ unsigned highs(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

}  // namespace duet
