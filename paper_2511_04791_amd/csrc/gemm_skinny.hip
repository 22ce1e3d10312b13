// Projections of few rows (decode steps) and the operators around them.
//
// A projection of n <= kSkinnyRows rows reads its whole weight matrix once and is bound by that
// read.  Weights are row-major [d_in, d_out] (output columns contiguous), so y^T = W^T x^T is
// computed: per 32 rows of W a wave takes 128 columns with eight 16-byte loads per lane (lane =
// 8 columns of row 8 (lane / 16) + r, 256 contiguous bytes per row), turns each lane's 8 x 8 block
// around in registers (32 byte permutes), and feeds eight 16x16x32 MFMAs per 16 rows of x: tile i
// takes every lane's column i.  x comes straight from the caches: the waves of a workgroup split
// d_in, so no wave shares its slice.  Workgroups cover (column tile, part of d_in); the waves of a
// workgroup add up through LDS, the parts through fp32 partials in the workspace, both in a
// fixed order that depends on the shape only.
//
// The kernel that adds the parts also runs the operator that follows, so nothing else passes over
// the rows: the output and down projections' adds the residual and normalises the new rows
// (residual_norm), the QKV projection's writes queries and cache (qkv_finish).  The gate-up
// projection's tiles pair 64 gate columns with the 64 up columns they meet and apply SwiGLU
// themselves.
//
// One layer of a decode-only step (Llama-3-8B sizes, contexts near 100): 16 rows 213 us with the
// library's products and separate operators, 116 us here; 64 rows 252 against 153 us; 70B sizes,
// 16 rows, 433 against 341 us.  The gate-up projection of 16 rows (235 MB) takes 47 us, 5.0 TB/s.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "wave_ops.h"

namespace duet {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kGWaves = 8;               // waves of a workgroup, each its own part of d_in
constexpr int kGThreads = 64 * kGWaves;
constexpr int kTileCols = 128;           // columns of W per workgroup
constexpr int kLdsStride = kTileCols + 4;

// Eight rows of W, 8 columns each (one lane's block of a step), and the lane's slice of x.
template <int NB>
struct Step {
  uint4 w[8];
  uint4 x[NB];
};

// Weights are read once and would push x out of the caches: non-temporal (4-7% on the whole chip).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 weight_load(const char* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// part[split][row][d_out] = x[rows, split's slice of d_in] W  (kSwiglu: gu and act, one split).
template <int NB, bool kSwiglu>
__global__ __launch_bounds__(kGThreads, 2) void skinny_gemm(SkinnyArgs a) {
  __shared__ __align__(16) float lds[kGWaves][16 * kLdsStride];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int c = lane & 15, quad = lane >> 4;
  const int tile = blockIdx.x % a.tiles, split = blockIdx.x / a.tiles;

  // The lane's 8 columns.  Lanes past the last column re-read column 0; nothing of theirs is stored.
  int col;
  if (kSwiglu) {
    const int g = tile * (kTileCols / 2) + 8 * (c & 7);
    col = g < a.m ? g + (c < 8 ? 0 : a.m) : 0;
  } else {
    col = tile * kTileCols + 8 * c;
    if (col >= a.d_out) col = 0;
  }
  // A load's address is a scalar base (the step's rows) plus the lane's 32-bit offset, fixed for the
  // whole loop.
  const unsigned w_lane = 2u * (8u * quad * a.d_out + col);
  unsigned x_lane[NB];  // rows past the last re-read it: their results are not stored
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) x_lane[nb] = 2u * (min(16 * nb + c, a.rows - 1) * (unsigned)a.d_in + 8u * quad);

  // The wave's steps of 32 rows of W; the last step of all may reach past d_in (a multiple of 8).
  const int steps = (a.d_in + 31) >> 5;
  const int parts = a.splits * kGWaves, part = split * kGWaves + wave;
  const int s0 = (int)((long long)steps * part / parts), s1 = (int)((long long)steps * (part + 1) / parts);
  auto load = [&](Step<NB>& st, int s) {
    const char* wb = reinterpret_cast<const char*>(a.w) + (size_t)(64u * (unsigned)s) * a.d_out;
    const char* xb = reinterpret_cast<const char*>(a.x) + 64u * (unsigned)s;
    const bool past = 32 * s + 8 * quad >= a.d_in;  // then read the step's first rows instead
    const unsigned wo = past ? 2u * col : w_lane;
#pragma unroll
    for (int r = 0; r < 8; ++r) st.w[r] = weight_load(wb + (size_t)(2u * r) * a.d_out + wo);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) st.x[nb] = *reinterpret_cast<const uint4*>(xb + (past ? x_lane[nb] - 16u * quad : x_lane[nb]));
    if (32 * s + 32 > a.d_in && past) {
#pragma unroll
      for (int r = 0; r < 8; ++r) st.w[r] = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) st.x[nb] = make_uint4(0, 0, 0, 0);
    }
  };
  f32x4 acc[8][NB];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const Step<NB>& st) {
    auto pair = [&](auto word, int i) {  // columns i and i + 1 of the block, rows 0 .. 7
      const uint4 lo = make_uint4(lows(word(0), word(1)), lows(word(2), word(3)), lows(word(4), word(5)), lows(word(6), word(7)));
      const uint4 hi = make_uint4(highs(word(0), word(1)), highs(word(2), word(3)), highs(word(4), word(5)), highs(word(6), word(7)));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const bf16x8 xf = __builtin_bit_cast(bf16x8, st.x[nb]);
        acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, lo), xf, acc[i][nb], 0, 0, 0);
        acc[i + 1][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, hi), xf, acc[i + 1][nb], 0, 0, 0);
      }
    };
    pair([&](int r) { return st.w[r].x; }, 0);
    pair([&](int r) { return st.w[r].y; }, 2);
    pair([&](int r) { return st.w[r].z; }, 4);
    pair([&](int r) { return st.w[r].w; }, 6);
  };
  // A ring of R steps in registers, all in flight until the oldest is multiplied (three and four
  // were 2-5% slower).  Loads are never branched on (steps past the last re-read it), so the wait
  // counts stay exact.
  constexpr int R = 2;
  Step<NB> ring[R];
  const int last = max(s1 - 1, 0);
#pragma unroll
  for (int u = 0; u < R; ++u) load(ring[u], min(s0 + u, last));
  int s = s0;
  for (; s + R < s1; s += R) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      multiply(ring[u]);
      load(ring[u], min(s + R + u, last));
    }
  }
#pragma unroll
  for (int u = 0; u < R; ++u)
    if (s + u < s1) multiply(ring[u]);

  // Sixteen rows at a time: acc[i][nb][r] is row 16 nb + lane % 16, column 8 (4 quad + r) + i.
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    if (16 * nb >= a.rows) break;
    if (nb > 0) __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float* p = &lds[wave][c * kLdsStride + 8 * (4 * quad + r)];
      *reinterpret_cast<f32x4*>(p) = f32x4{acc[0][nb][r], acc[1][nb][r], acc[2][nb][r], acc[3][nb][r]};
      *reinterpret_cast<f32x4*>(p + 4) = f32x4{acc[4][nb][r], acc[5][nb][r], acc[6][nb][r], acc[7][nb][r]};
    }
    __syncthreads();
    auto sum4 = [&](int row, int at) {
      f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < kGWaves; ++v) t += *reinterpret_cast<const f32x4*>(&lds[v][row * kLdsStride + at]);
      return t;
    };
    if (kSwiglu) {
      const int row = tid >> 4, at = 4 * (tid & 15);  // the first 256 threads
      const int g = tile * (kTileCols / 2) + at;
      if (tid < 256 && 16 * nb + row < a.rows && g < a.m) {
        const f32x4 gs = sum4(row, at), us = sum4(row, kTileCols / 2 + at);
        bf16x4 gb, ub, o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          gb[e] = static_cast<__bf16>(gs[e]);
          ub[e] = static_cast<__bf16>(us[e]);
          const float gf = static_cast<float>(gb[e]);
          o[e] = static_cast<__bf16>(gf / (1.0f + expf(-gf)) * static_cast<float>(ub[e]));
        }
        const size_t r = 16 * nb + row;
        *reinterpret_cast<bf16x4*>(a.gu + r * 2 * a.m + g) = gb;
        *reinterpret_cast<bf16x4*>(a.gu + r * 2 * a.m + a.m + g) = ub;
        *reinterpret_cast<bf16x4*>(a.act + r * a.m + g) = o;
      }
    } else {
      const int row = tid >> 5, at = 4 * (tid & 31);
      const int cc = tile * kTileCols + at;
      if (16 * nb + row < a.rows && cc < a.d_out)
        *reinterpret_cast<f32x4*>(a.part + ((size_t)split * a.rows + 16 * nb + row) * a.d_out + cc) = sum4(row, at);
    }
  }
}

__device__ __forceinline__ f32x4 sum_parts(const float* p, int splits, size_t stride) {
  f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int s = 0; s < splits; ++s) t += *reinterpret_cast<const f32x4*>(p + s * stride);
  return t;
}

// One workgroup per row: x = bf16(x + sum of the parts), then y = RMSNorm(x) * w (no norm without w).
__global__ __launch_bounds__(1024) void residual_norm(const float* part, int splits, __bf16* x, const __bf16* w,
                                                      __bf16* y, int rows, int d, float eps) {
  __shared__ float red[16];
  const size_t row = blockIdx.x;
  __bf16* xr = x + row * d;
  const float* pr = part + row * d;
  float ss = 0.f;
  for (int e = 4 * threadIdx.x; e < d; e += 4 * blockDim.x) {
    const bf16x4 old = *reinterpret_cast<const bf16x4*>(xr + e);
    const f32x4 t = sum_parts(pr + e, splits, (size_t)rows * d);
    bf16x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = static_cast<__bf16>(static_cast<float>(old[i]) + t[i]);
      const float f = static_cast<float>(v[i]);
      ss += f * f;
    }
    *reinterpret_cast<bf16x4*>(xr + e) = v;
  }
  if (!w) return;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = 0.f;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) ss += red[i];
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int e = 4 * threadIdx.x; e < d; e += 4 * blockDim.x) {  // each thread re-reads what it wrote
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(xr + e), g = *reinterpret_cast<const bf16x4*>(w + e);
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = static_cast<__bf16>(static_cast<float>(v[i]) * inv * static_cast<float>(g[i]));
    *reinterpret_cast<bf16x4*>(y + row * d + e) = o;
  }
}

// Four columns of one row per thread: qkv = bf16(sum of the parts), then the QKV split of the row.
__global__ __launch_bounds__(256) void qkv_finish(const float* part, int splits, __bf16* qkv, QkvSplitArgs s) {
  const int nq = s.h_q * s.head_dim, nk = s.h_kv * s.head_dim, width = nq + 2 * nk;
  const int i = blockIdx.y;
  const int col = 4 * (blockIdx.x * 256 + threadIdx.x);
  const int row = s.row0 + i;
  // The row's request (whole waves search), then the page and slot of its position.
  const int r = s.dreq ? s.dreq[row].x : find_request(s.num_reqs, [&](int x) { return s.meta[x].y <= row; });
  const int4 m = s.meta[r];
  const int pos = s.dreq ? m.w : m.w + (row - m.y);
  const int id = s.page_table[(size_t)r * s.max_pages + (pos >> 4)], slot = pos & 15;
  if (col >= width) return;
  const f32x4 t = sum_parts(part + (size_t)i * width + col, splits, (size_t)s.rows * width);
  bf16x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = static_cast<__bf16>(t[e]);
  *reinterpret_cast<bf16x4*>(qkv + (size_t)i * width + col) = v;
  if (col < nq) {
    *reinterpret_cast<bf16x4*>(s.q + (size_t)row * nq + col) = v;
    return;
  }
  if (!page_ok(id, s.num_phys_pages)) {
    if (col == nq) atomicOr(s.err, 1);
    return;
  }
  const int kv = col - nq;
  const int j = (kv % nk) / s.head_dim, e0 = kv % s.head_dim;
  const size_t slab = (size_t)id * s.h_kv + j;
  if (kv < nk) {
    *reinterpret_cast<bf16x4*>(s.k_cache + (slab * 16 + slot) * s.head_dim + e0) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) s.v_cache[(slab * s.head_dim + e0 + e) * 16 + slot] = v[e];
  }
}

template <bool kSwiglu>
hipError_t launch(const SkinnyArgs& a, hipStream_t s) {
  const dim3 grid(a.tiles * a.splits), block(kGThreads);
  if (a.rows <= 16) hipLaunchKernelGGL((skinny_gemm<1, kSwiglu>), grid, block, 0, s, a);
  else if (a.rows <= 32) hipLaunchKernelGGL((skinny_gemm<2, kSwiglu>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((skinny_gemm<4, kSwiglu>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace

bool use_skinny(int rows, int cus, int d, int d_qkv, int m, size_t bytes) {
  const int widest = std::max(d, d_qkv);
  if (rows < 1 || rows > kSkinnyRows || (size_t)rows * widest * sizeof(float) > bytes) return false;
  const bool whole = cus == DUET_TOTAL_CUS;
  const size_t weights = (size_t)d * (d_qkv + d + 3 * (size_t)m) * sizeof(__bf16);
  // Rows (of whole tiles) times weights that a share of `cus` CUs takes.
  const size_t most = (size_t)18000000 * std::min(cus, 128);
  if (rows > kSkinnyRows / 2) {
    const bool narrow = widest <= 1536;
    return whole ? narrow || m >= 2 * d : narrow && kSkinnyRows * weights <= most;
  }
  if (whole) return true;
  if (cus >= 96) return weights <= (size_t)512 << 20;
  return weights <= (size_t)64 << 20 && (rows <= 16 ? 16 : 32) * weights <= most;
}

// Parts of d_in: about one workgroup per CU of the whole chip, each wave with a step of its own, partials
// within `bytes`.  Never per share: every share that takes these kernels adds in the same order.
int skinny_splits(int rows, int d_in, int d_out, size_t bytes) {
  const int tiles = (d_out + kTileCols - 1) / kTileCols;
  const int steps = (d_in + 31) / 32;
  const long long fit = (long long)(bytes / ((size_t)rows * d_out * sizeof(float)));
  return (int)std::max<long long>(1, std::min<long long>({256 / tiles, steps / kGWaves, 16, fit}));
}

hipError_t launch_skinny_gemm(const __bf16* x, const __bf16* w, float* part, int rows, int d_in, int d_out, int splits,
                              hipStream_t s) {
  SkinnyArgs a{};
  a.x = x;
  a.w = w;
  a.part = part;
  a.rows = rows;
  a.d_in = d_in;
  a.d_out = d_out;
  a.splits = splits;
  a.tiles = (d_out + kTileCols - 1) / kTileCols;
  return launch<false>(a, s);
}

hipError_t launch_skinny_gate_up(const __bf16* x, const __bf16* w, __bf16* gu, __bf16* act, int rows, int d_in, int m,
                                 hipStream_t s) {
  SkinnyArgs a{};
  a.x = x;
  a.w = w;
  a.gu = gu;
  a.act = act;
  a.rows = rows;
  a.d_in = d_in;
  a.d_out = 2 * m;
  a.m = m;
  a.splits = 1;
  a.tiles = (m + kTileCols / 2 - 1) / (kTileCols / 2);
  return launch<true>(a, s);
}

hipError_t launch_residual_norm(const float* part, int splits, __bf16* x, const __bf16* w, __bf16* y, int rows, int d,
                                float eps, hipStream_t s) {
  const int threads = std::min(1024, (d / 4 + 63) / 64 * 64);
  hipLaunchKernelGGL(residual_norm, dim3(rows), dim3(threads), 0, s, part, splits, x, w, y, rows, d, eps);
  return hipGetLastError();
}

hipError_t launch_qkv_finish(const float* part, int splits, __bf16* qkv, const QkvSplitArgs& a, hipStream_t s) {
  const int width = (a.h_q + 2 * a.h_kv) * a.head_dim;
  hipLaunchKernelGGL(qkv_finish, dim3((width + 1023) / 1024, a.rows), dim3(256), 0, s, part, splits, qkv, a);
  return hipGetLastError();
}

}  // namespace duet
