// fp32 attention over the paged KV cache: prefill chunks and the decode split-K partials.
//
// Both kernels walk 16-token pages with one body (f32_page), on the fp32 MFMA (16x16x4):
//   S^T [16 tokens x 16 columns]  = K_page [16 x d] . Q^T [d x 16]
//   O^T [d x 16 columns]         += V_page^T [d x 16] . P^T [16 x 16]
// A column is one (query row, query head): 16 consecutive queries of a head for prefill, the
// query heads of the GQA group for decode (columns past the group are zero).  K and V pages are
// read with 16 bytes per lane; the MFMA's four contraction slots of a step take components
// 0 .. 3 of those words (the order of a contraction is free as long as both operands agree), so
// a score register holds exactly the token whose V word it multiplies and P^T never leaves the
// lane.
//
// What bounds these kernels is latency, not bytes or FLOPs (fp32 is for small shapes).  The row
// of work is therefore cut fine: a prefill workgroup owns 16 queries of one head and its eight
// waves take every eighth page, then merge through LDS; a decode wave owns two pages.  A
// 48-token chunk after 16 tokens, 4 heads of 64, went from 398 us (a wave walked 32 rows key by
// key, one shuffle reduction per key) to 4.9 us, and its decode partials (contexts 17 .. 100) from
// 24 us to 5.0 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "wave_ops.h"

namespace duet {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Waves = 8;  // waves per prefill workgroup
constexpr int kF32Rows = 16;  // queries per prefill workgroup

// One page of one kv head.  k: token lane % 16, dims 16 s + 4 (lane / 16) + 0..3.
// v: dim 16 n + lane % 16, tokens 4 (lane / 16) + 0..3.
template <int D>
struct F32Page {
  f32x4 k[D / 16], v[D / 16];
  bool ok;
};

template <int D>
__device__ __forceinline__ size_t slab_of(const F32Page<D>& pg, const AttnArgs& a, int id, int j) {
  return ((size_t)(pg.ok ? id : 0) * a.h_kv + j) * 16 * D;
}
template <int D>
__device__ __forceinline__ void load_k(F32Page<D>& pg, const AttnArgs& a, int id, int j, int lane) {
  pg.ok = page_ok(id, a.num_phys_pages);
  const float* kp = reinterpret_cast<const float*>(a.k_cache) + slab_of(pg, a, id, j) + (lane & 15) * D + 4 * (lane >> 4);
#pragma unroll
  for (int s = 0; s < D / 16; ++s) pg.k[s] = *reinterpret_cast<const f32x4*>(kp + 16 * s);
}
template <int D>
__device__ __forceinline__ void load_v(F32Page<D>& pg, const AttnArgs& a, int id, int j, int lane) {
  const float* vp = reinterpret_cast<const float*>(a.v_cache) + slab_of(pg, a, id, j) + (lane & 15) * 16 + 4 * (lane >> 4);
#pragma unroll
  for (int n = 0; n < D / 16; ++n) pg.v[n] = *reinterpret_cast<const f32x4*>(vp + 256 * n);
}

// Running softmax state of a wave's 16 columns (column = lane % 16): reference max in base-2
// units (shared by the column's four lanes), this lane's part of the denominator, and the
// unnormalised output, dims 16 n + 4 (lane / 16) + r in acc[n][r].
template <int D>
struct F32State {
  float m = -INFINITY, l = 0.f;
  f32x4 acc[D / 16];
  __device__ F32State() {
#pragma unroll
    for (int n = 0; n < D / 16; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
};

// Adds page p (tokens 16 p .. 16 p + 15).  A column sees tokens 0 .. last (its own bound); tokens
// n_tok and later are not part of the request and may hold anything.  kCausal: last differs
// between columns, so a token can be hidden from one column and seen by another.
template <int D, bool kCausal>
__device__ __forceinline__ void f32_page(F32State<D>& st, const F32Page<D>& pg, const f32x4 (&q)[D / 16], int p,
                                         int last, int n_tok, const AttnArgs& a, int id, int j, int lane) {
  if (!pg.ok) return;  // flagged by the caller; its tokens do not exist
  const int quad = lane >> 4;
  const int t0 = 16 * p + 4 * quad;
  // Four accumulators: independent MFMA chains, and shorter sums.
  f32x4 part[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) part[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(pg.k[s][i], q[s][i], part[i], 0, 0, 0);
  float x[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float dot = (part[0][r] + part[1][r]) + (part[2][r] + part[3][r]);
    x[r] = t0 + r <= last ? dot * a.scale_log2 : -INFINITY;
  }
  const float mx = max_rows(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
  const float m_new = fmaxf(st.m, mx);
  const float m_sub = m_new == -INFINITY ? 0.f : m_new;  // no token yet: every weight is 2^-inf = 0
  const float alpha = fast_exp2(st.m - m_sub);
  st.m = m_new;
  float pr[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) pr[r] = fast_exp2(x[r] - m_sub);
  st.l = st.l * alpha + ((pr[0] + pr[1]) + (pr[2] + pr[3]));
#pragma unroll
  for (int n = 0; n < D / 16; ++n) st.acc[n] *= alpha;
  if (kCausal && 16 * p + 15 > __builtin_amdgcn_readfirstlane(last)) {
    // A page on the diagonal: a value hidden from some columns meets their zero weights in the
    // MFMA, which is only harmless if it is finite.  The values of such a page that are not are
    // kept away from those columns by adding its tokens one by one.
    float z = 0.f;
#pragma unroll
    for (int n = 0; n < D / 16; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (t0 + r < n_tok) z += pg.v[n][r] * 0.f;
    if (__any(z != 0.f)) {
      const float* vp = reinterpret_cast<const float*>(a.v_cache) + ((size_t)id * a.h_kv + j) * 16 * D;
#pragma unroll 1
      for (int t = 0; t < 16; ++t) {
        const int i = t & 3;
        const float w = __shfl(i < 2 ? (i == 0 ? pr[0] : pr[1]) : (i == 2 ? pr[2] : pr[3]), (lane & 15) + 16 * (t >> 2));
        if (16 * p + t > last) continue;
#pragma unroll
        for (int n = 0; n < D / 16; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) st.acc[n][r] += w * vp[(16 * n + 4 * quad + r) * 16 + t];
      }
      return;
    }
  }
  const bool tail = 16 * (p + 1) > n_tok;
#pragma unroll
  for (int n = 0; n < D / 16; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = tail && t0 + r >= n_tok ? 0.f : pg.v[n][r];
      st.acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, pr[r], st.acc[n], 0, 0, 0);
    }
}

// Sixteen queries of one head per workgroup; workgroup b is row block b % 8 of item b / 8.
template <int D>
__global__ __launch_bounds__(64 * kF32Waves) void prefill_f32(AttnArgs a, WorkArgs w) {
  constexpr int kStride = D + 4;  // floats per column in LDS: columns start on different banks
  __shared__ __align__(16) float part[kF32Waves][kF32Rows * kStride];
  __shared__ float ml[kF32Waves][2][kF32Rows];
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, quad = lane >> 4;
  constexpr int kBlocks = kPrefillRows / kF32Rows;
  const PrefillItem it = w.pitems[blockIdx.x / kBlocks];
  const int r = it.req, h = it.head, row0 = it.row0 + kF32Rows * (blockIdx.x % kBlocks);
  const int q_start = it.q_start, q_len = it.q_len, c = it.cached_len;
  if (row0 >= q_len) return;
  const int j = h / a.group;
  const int qi = row0 + col;
  const bool row_ok = qi < q_len;
  const int n_tok = c + q_len;
  const int n_pages = (c + min(row0 + kF32Rows, q_len) - 1) / 16 + 1;

  f32x4 q[D / 16];
  {
    const float* qp = reinterpret_cast<const float*>(a.q) + ((size_t)(q_start + (row_ok ? qi : row0)) * a.h_q + h) * D +
                      4 * quad;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) q[s] = *reinterpret_cast<const f32x4*>(qp + 16 * s);
  }
  F32State<D> st;
  const int* prow = a.page_table + (size_t)r * a.max_pages;
  bool bad = false;
  // Pages wave, wave + 8, ...; their ids are fetched 64 at a time, one per lane.
  for (int p0 = wave; p0 < n_pages; p0 += 64 * kF32Waves) {
    const int n_here = min(64, (n_pages - p0 + kF32Waves - 1) / kF32Waves);
    const int ids = lane < n_here ? prow[p0 + kF32Waves * lane] : 0;
    // A page's values and the next page's keys load while its scores are computed.
    F32Page<D> pg;
    load_k<D>(pg, a, __builtin_amdgcn_readlane(ids, 0), j, lane);
    for (int i = 0; i < n_here; ++i) {
      const int id = __builtin_amdgcn_readlane(ids, i);
      load_v<D>(pg, a, id, j, lane);
      F32Page<D> nx;
      load_k<D>(nx, a, __builtin_amdgcn_readlane(ids, min(i + 1, n_here - 1)), j, lane);
      bad |= !pg.ok;
      f32_page<D, true>(st, pg, q, p0 + kF32Waves * i, c + qi, n_tok, a, id, j, lane);
      pg = nx;
    }
  }
  if (bad && lane == 0) atomicOr(w.err, 1);

  // Merge of the eight waves: weights against the common max, sums in wave order.
  const float l = sum_rows(st.l);
#pragma unroll
  for (int n = 0; n < D / 16; ++n)
    *reinterpret_cast<f32x4*>(&part[wave][col * kStride + 16 * n + 4 * quad]) = st.acc[n];
  if (quad == 0) {
    ml[wave][0][col] = st.m;
    ml[wave][1][col] = l;
  }
  __syncthreads();
  float* out = reinterpret_cast<float*>(a.out);
  for (int x = threadIdx.x; x < kF32Rows * D / 4; x += 64 * kF32Waves) {
    const int cc = x / (D / 4), e = 4 * (x % (D / 4));
    if (row0 + cc >= q_len) continue;
    float mm = -INFINITY;
#pragma unroll
    for (int v = 0; v < kF32Waves; ++v) mm = fmaxf(mm, ml[v][0][cc]);
    float den = 0.f;
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < kF32Waves; ++v) {
      if (v >= n_pages) break;  // waves without a page
      const float wgt = fast_exp2(ml[v][0][cc] - mm);
      den += wgt * ml[v][1][cc];
      num += wgt * *reinterpret_cast<const f32x4*>(&part[v][cc * kStride + e]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) num[i] /= den;
    *reinterpret_cast<f32x4*>(out + ((size_t)(q_start + row0 + cc) * a.h_q + h) * D + e) = num;
  }
}

// One wave per (request, kv head, split of kDecodePagesPerSplitF32 pages).
template <int D>
__global__ __launch_bounds__(256) void decode_partial_f32(AttnArgs a, WorkArgs w) {
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, quad = lane >> 4;
  const int4 dr = w.dreq[blockIdx.y];
  const int witem = blockIdx.x * 4 + wave;
  const int j = witem / dr.z;
  const int s = witem - j * dr.z;
  if (j >= a.h_kv) return;
  const int4 m = w.meta[dr.x];
  const int n_tok = m.w + m.z;
  const int g = a.group;
  const int pb = s * kDecodePagesPerSplitF32;
  const int pe = min(pb + kDecodePagesPerSplitF32, dr.w);
  const int* prow = a.page_table + (size_t)dr.x * a.max_pages;
  const int item = dr.y + j * dr.z + s;
  f32x4 q[D / 16];
  {
    const float* qp = reinterpret_cast<const float*>(a.q) + ((size_t)m.y * a.h_q + j * g + min(col, g - 1)) * D + 4 * quad;
#pragma unroll
    for (int x = 0; x < D / 16; ++x) q[x] = *reinterpret_cast<const f32x4*>(qp + 16 * x);
  }
  F32State<D> st;
  bool bad = false;
  int id = uniform(prow[pb]);
  F32Page<D> pg;
  load_k<D>(pg, a, id, j, lane);
  load_v<D>(pg, a, id, j, lane);
  for (int p = pb; p < pe; ++p) {
    const int id_n = uniform(prow[min(p + 1, pe - 1)]);
    F32Page<D> nx;
    load_k<D>(nx, a, id_n, j, lane);
    load_v<D>(nx, a, id_n, j, lane);
    bad |= !pg.ok;
    f32_page<D, false>(st, pg, q, p, n_tok - 1, n_tok, a, id, j, lane);
    pg = nx;
    id = id_n;
  }
  const float l = sum_rows(st.l);
  if (col < g) {
    float* pa = w.pacc + ((size_t)item * g + col) * D + 4 * quad;
#pragma unroll
    for (int n = 0; n < D / 16; ++n) *reinterpret_cast<f32x4*>(pa + 16 * n) = st.acc[n];
    if (quad == 0) {
      w.pml[((size_t)item * g + col) * 2 + 0] = st.m;
      w.pml[((size_t)item * g + col) * 2 + 1] = l;
    }
  }
  if (bad && lane == 0) atomicOr(w.err, 1);
}

}  // namespace

hipError_t launch_decode_partial_f32(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  const dim3 grid((a.h_kv * w.max_split + 3) / 4, w.n_dreq);
  if (a.head_dim == 128) hipLaunchKernelGGL(decode_partial_f32<128>, grid, dim3(256), 0, s, a, w);
  else hipLaunchKernelGGL(decode_partial_f32<64>, grid, dim3(256), 0, s, a, w);
  return hipGetLastError();
}

hipError_t launch_prefill_f32(const AttnArgs& a, const WorkArgs& w, hipStream_t s) {
  constexpr int kBlocks = kPrefillRows / kF32Rows, kThreads = 64 * kF32Waves;
  constexpr int kItems = 1 << 19;  // of one launch: a grid holds fewer than 2^32 threads
  static_assert((unsigned long long)kItems * kBlocks * kThreads < 1ULL << 32, "a launch fits");
  for (int i0 = 0; i0 < w.n_pitems; i0 += kItems) {
    WorkArgs part = w;
    part.pitems += i0;
    const dim3 grid(std::min(kItems, w.n_pitems - i0) * kBlocks);
    if (a.head_dim == 128) hipLaunchKernelGGL(prefill_f32<128>, grid, dim3(kThreads), 0, s, a, part);
    else hipLaunchKernelGGL(prefill_f32<64>, grid, dim3(kThreads), 0, s, a, part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace duet
