// Token-level operators of a transformer block (paper, Section 4.1, "Token-Level Operators"):
// RMSNorm, the SwiGLU activation, and the step between the QKV projection and attention that
// takes the query rows out of the projection and writes the new tokens' keys and values into the
// paged cache (Section 2: a token's key and value are appended before attention reads them).
// The projections themselves are plain GEMMs (hipBLASLt, issued by the runtime).
//
// All three are HBM-bound elementwise passes over [rows, width] bf16 activations: 16-byte
// accesses, fp32 arithmetic, round-to-nearest-even on store.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "wave_ops.h"

namespace duet {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
  return t;
}

// y[r] = x[r] / sqrt(mean(x[r]^2) + eps) * w, for rows r of [rows, d] (d a multiple of 8).  U > 0: a
// thread keeps its (at most U) 8-value chunks of the row between the sum and the scaling; U = 0 (rows
// too long for that) reads the row twice.
template <int U>
__global__ __launch_bounds__(256) void rmsnorm_bf16(const __bf16* x, const __bf16* w, __bf16* y, int d, float eps) {
  __shared__ float red[4];
  const size_t row = blockIdx.x;
  const bf16x8* xr = reinterpret_cast<const bf16x8*>(x + row * d);
  const bf16x8* wr = reinterpret_cast<const bf16x8*>(w);
  bf16x8* yr = reinterpret_cast<bf16x8*>(y + row * d);
  const int n = d / 8;
  auto squares = [](const bf16x8& v, float ss) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float f = static_cast<float>(v[e]);
      ss += f * f;
    }
    return ss;
  };
  auto scaled = [](const bf16x8& v, const bf16x8& g, float inv) {
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(static_cast<float>(v[e]) * inv * static_cast<float>(g[e]));
    return o;
  };
  float ss = 0.f;
  if constexpr (U > 0) {
    bf16x8 v[U], g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = min((int)threadIdx.x + 256 * u, n - 1);
      v[u] = xr[c];
      g[u] = wr[c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((int)threadIdx.x + 256 * u < n) ss = squares(v[u], ss);
    const float inv = 1.0f / sqrtf(block_sum(ss, red) / (float)d + eps);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((int)threadIdx.x + 256 * u < n) yr[threadIdx.x + 256 * u] = scaled(v[u], g[u], inv);
  } else {
    for (int c = threadIdx.x; c < n; c += 256) ss = squares(xr[c], ss);
    const float inv = 1.0f / sqrtf(block_sum(ss, red) / (float)d + eps);
    for (int c = threadIdx.x; c < n; c += 256) yr[c] = scaled(xr[c], wr[c], inv);
  }
}

// a[r, i] = silu(gu[r, i]) * gu[r, m + i]: gate columns first, then up (m a multiple of 8).  A thread
// takes kSwigluChunks 8-value chunks of a row, 256 apart, all loaded before the first is used.
constexpr int kSwigluChunks = 2;
__global__ __launch_bounds__(256) void swiglu_bf16(const __bf16* gu, __bf16* a, int m, int blocks_per_row) {
  const size_t row = blockIdx.x / blocks_per_row;
  const int c0 = (blockIdx.x % blocks_per_row) * 256 * kSwigluChunks + threadIdx.x;
  const bf16x8* g = reinterpret_cast<const bf16x8*>(gu + row * 2 * m);
  const bf16x8* u = reinterpret_cast<const bf16x8*>(gu + row * 2 * m + m);
  bf16x8* o = reinterpret_cast<bf16x8*>(a + row * m);
  const int n = m / 8;
  bf16x8 gv[kSwigluChunks], uv[kSwigluChunks];
#pragma unroll
  for (int k = 0; k < kSwigluChunks; ++k) {
    const int c = min(c0 + 256 * k, n - 1);
    gv[k] = g[c];
    uv[k] = u[c];
  }
#pragma unroll
  for (int k = 0; k < kSwigluChunks; ++k) {
    if (c0 + 256 * k >= n) break;
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float gf = static_cast<float>(gv[k][e]);
      r[e] = static_cast<__bf16>(gf / (1.0f + expf(-gf)) * static_cast<float>(uv[k][e]));
    }
    o[c0 + 256 * k] = r;
  }
}

// The QKV projection [rows, (h_q + 2 h_kv) d] of the launch's rows: query columns to q (row stride
// h_q d), key and value columns to the slots of their positions in the paged cache.
//
// A workgroup takes the rows of one request whose positions lie on one page (up to 16; one decode row)
// and 2048 columns, a thread 8 columns of all of them.  Queries and keys are copied 16 bytes at a
// time.  Values go to a dim-major page: the 8 x 16 block of a whole page is turned around in
// registers (byte permutes) and each dim's 16 tokens written as 32 contiguous bytes; of a page that
// the chunk covers in part, value by value.  Writing every value alone, one workgroup per row, took
// 31.6 us on 2112 rows of 6144 columns (52 MB moved); this takes 18.0 us (in a block, where the
// projection is still in the caches, 23.8 and 12.5 us).
//
// Request r (rows q_start .. q_start + q_len - 1) has the page groups from q_start / 16 + 2 r on: more
// than it needs, whatever its first slot, and groups past its last page end at once.  In a look-ahead
// step (dreq) group b is row b, the token of decode request b at the step's cached_len.  A page id
// outside [0, num_phys_pages) is not written through: it sets bit 0 of the error word.
__device__ __forceinline__ int first_group(const QkvSplitArgs& s, int r) { return (s.meta[r].y >> 4) + 2 * r; }

__global__ __launch_bounds__(256) void qkv_split_bf16(QkvSplitArgs s) {
  const int nq = s.h_q * s.head_dim, nk = s.h_kv * s.head_dim, width = nq + 2 * nk, d = s.head_dim;
  const int group = blockIdx.x;
  int r, row, n, pos;  // request, first row, rows, position of the first row
  if (s.dreq) {
    r = s.dreq[group].x;
    row = group;
    n = 1;
    pos = s.meta[r].w;
  } else {
    r = uniform(find_request(s.num_reqs, [&](int x) { return first_group(s, x) <= group; }));
    const int4 m = s.meta[r];
    if (m.y < s.row0 || m.y >= s.row0 + s.rows) return;  // another partition's request
    const int page = (m.w >> 4) + group - ((m.y >> 4) + 2 * r);
    pos = max(m.w, 16 * page);
    n = min(m.w + m.z, 16 * page + 16) - pos;
    if (n <= 0) return;
    row = m.y + pos - m.w;
  }
  const int col = 8 * (blockIdx.y * 256 + threadIdx.x);
  if (col >= width) return;
  const int id = s.page_table[(size_t)r * s.max_pages + (pos >> 4)];
  const int slot = pos & 15;
  if (col >= nq && !page_ok(id, s.num_phys_pages)) {
    if (col == nq) atomicOr(s.err, 1);
    return;
  }
  // Every row is loaded before the first store (rows past the last re-read it): one memory latency
  // for the group, which is what a page covered in part costs too.
  const __bf16* src = s.qkv + (size_t)row * width + col;
  uint4 x[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) x[t] = *reinterpret_cast<const uint4*>(src + (size_t)min(t, n - 1) * width);
  if (col < nq + nk) {
    __bf16* dst;
    size_t stride;
    if (col < nq) {
      dst = s.q + (size_t)row * nq + col;
      stride = nq;
    } else {
      dst = s.k_cache + (((size_t)id * s.h_kv + (col - nq) / d) * 16 + slot) * d + (col - nq) % d;
      stride = d;
    }
#pragma unroll
    for (int t = 0; t < 16; ++t)
      if (t < n) *reinterpret_cast<uint4*>(dst + t * stride) = x[t];
    return;
  }
  const int kv = col - nq - nk;
  __bf16* v = s.v_cache + (((size_t)id * s.h_kv + kv / d) * d + kv % d) * 16 + slot;
  if (n < 16) {
#pragma unroll
    for (int t = 0; t < 16; ++t)
      if (t < n) {
        const bf16x8 y = __builtin_bit_cast(bf16x8, x[t]);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i * 16 + t] = y[i];
      }
    return;
  }
  auto turn = [&](auto word, int i) {  // dims i and i + 1 of a whole page
    unsigned lo[8], hi[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      lo[t] = lows(word(x[2 * t]), word(x[2 * t + 1]));
      hi[t] = highs(word(x[2 * t]), word(x[2 * t + 1]));
    }
    uint4* p = reinterpret_cast<uint4*>(v + i * 16);
    p[0] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    p[1] = make_uint4(lo[4], lo[5], lo[6], lo[7]);
    p[2] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    p[3] = make_uint4(hi[4], hi[5], hi[6], hi[7]);
  };
  turn([](const uint4& w) { return w.x; }, 0);
  turn([](const uint4& w) { return w.y; }, 2);
  turn([](const uint4& w) { return w.z; }, 4);
  turn([](const uint4& w) { return w.w; }, 6);
}

}  // namespace

hipError_t launch_rmsnorm(const __bf16* x, const __bf16* w, __bf16* y, int rows, int d, float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const dim3 grid(rows), block(256);
  if (d <= 2048) hipLaunchKernelGGL(rmsnorm_bf16<1>, grid, block, 0, s, x, w, y, d, eps);
  else if (d <= 4096) hipLaunchKernelGGL(rmsnorm_bf16<2>, grid, block, 0, s, x, w, y, d, eps);
  else if (d <= 8192) hipLaunchKernelGGL(rmsnorm_bf16<4>, grid, block, 0, s, x, w, y, d, eps);
  else hipLaunchKernelGGL(rmsnorm_bf16<0>, grid, block, 0, s, x, w, y, d, eps);
  return hipGetLastError();
}

hipError_t launch_swiglu(const __bf16* gu, __bf16* a, int rows, int m, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int per_row = (m / 8 + 256 * kSwigluChunks - 1) / (256 * kSwigluChunks);
  const int most = (int)(((1u << 24) - 1) / per_row);  // rows of one launch: a grid holds fewer than 2^32 threads
  for (int r0 = 0; r0 < rows; r0 += std::min(most, rows - r0)) {
    hipLaunchKernelGGL(swiglu_bf16, dim3(std::min(most, rows - r0) * per_row), dim3(256), 0, s, gu + (size_t)r0 * 2 * m,
                       a + (size_t)r0 * m, m, per_row);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_qkv_split(const QkvSplitArgs& a, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  const int width = (a.h_q + 2 * a.h_kv) * a.head_dim;
  // Every request's groups up to the launch's last row (first_group of the request after it).
  const int groups = a.dreq ? a.rows : (a.row0 + a.rows) / 16 + 2 * a.num_reqs;
  hipLaunchKernelGGL(qkv_split_bf16, dim3(groups, (width / 8 + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace duet
