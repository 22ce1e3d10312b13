// Device code of the bf16 decode kernels (attn_decode.hip says what it computes and how).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"
#include "wave_ops.h"

namespace duet {
namespace decode {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr float kRescaleSlack = 8.0f;  // base-2 units: probabilities stay below 2^8
constexpr int kRing = 4;  // page buffers per wave: kRing - 1 pages in flight
typedef float f32x4 __attribute__((ext_vector_type(4)));


// K/V pages are read exactly once per iteration (plain loads: non-temporal loads were measured
// slower under the split).
template <typename T>
__device__ __forceinline__ T stream_load(const char* p) {
  return *reinterpret_cast<const T*>(p);
}

__device__ __forceinline__ uint64_t low_elems_mask(int n) {  // keep the first n of 4 bf16
  return n >= 4 ? ~0ull : (n <= 0 ? 0ull : ((1ull << (16 * n)) - 1ull));
}

template <int D>
struct Page {
  uint4 k[D / 32];  // K rows (token = lane % 16), 8 dims per lane per 32-dim step
  uint2 v[D / 16];  // V^T rows (dim = 16 n + lane % 16), tokens 4 (lane / 16) .. +4
};

template <int D>
__device__ __forceinline__ void load_k(Page<D>& pg, const char* kbase, size_t slab, int lane) {
  constexpr size_t kPageBytes = 16 * D * 2;  // one (page, kv head) slab
  const char* kp = kbase + slab * kPageBytes + (lane & 15) * D * 2 + (lane >> 4) * 16;
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) pg.k[ks] = stream_load<uint4>(kp + ks * 64);
}
template <int D>
__device__ __forceinline__ void load_v(Page<D>& pg, const char* vbase, size_t slab, int lane) {
  constexpr size_t kPageBytes = 16 * D * 2;
  const char* vp = vbase + slab * kPageBytes + (lane & 15) * 32 + (lane >> 4) * 8;
#pragma unroll
  for (int n = 0; n < D / 16; ++n) pg.v[n] = stream_load<uint2>(vp + n * 16 * 32);
}
template <int D>
__device__ __forceinline__ void load_page(Page<D>& pg, const char* kbase, const char* vbase, size_t slab, int lane) {
  load_k<D>(pg, kbase, slab, lane);
  load_v<D>(pg, vbase, slab, lane);
}

// Uniform loads of the read-only work list through the scalar cache (used before the page stream
// starts; inside it a scalar load would be waited for together with every LDS operation).
__device__ __forceinline__ i32x4 sload4(const void* p) { return *(const __attribute__((address_space(4))) i32x4*)(p); }

// A decode work item as the host lists it: (q_start, req | kv head << 24, first page |
// (tokens - 1) << 22, row of its split-K partial).  The item covers `tokens` keys (at most 16 PPS)
// from its first logical page on.
struct DItem {
  int q_start, req, j, first_page, n_tok, slot;
  bool valid;
};
__device__ __forceinline__ DItem unpack_item(i32x4 v, bool valid) {
  DItem d;
  d.q_start = v.x;
  d.req = v.y & 0xffffff;
  d.j = (int)((unsigned)v.y >> 24);
  d.first_page = v.z & 0x3fffff;
  d.n_tok = (int)((unsigned)v.z >> 22) + 1;
  d.slot = v.w;
  d.valid = valid;
  return d;
}

// Merges the splits of one (decode request, query head) pair, pair = request * h_q + head, with
// one wave.  Lanes first take one split each to find the common max and the denominator, then take
// one dim each to sum the weighted outputs.
template <int D, typename OutT>
__device__ __forceinline__ void merge_pair(const AttnArgs& a, const WorkArgs& w, const float* pacc, const float* pml,
                                           void* out, int pair, int lane) {
  constexpr int E = D / 64;
  const int i = pair / a.h_q;
  const int h = pair - i * a.h_q;
  const int4 dr = w.dreq[i];
  const int g = a.group;
  const int j = h / g, col = h - j * g;
  const size_t base = (size_t)(dr.y + j * dr.z) * g + col;  // partial row of split 0
  const int n = dr.z;
  // Eight partial rows (splits s0 + t0 .. + 7 of the cnt from s0) are loaded before any is used,
  // so their loads overlap.
  float part[8][E];
  auto load_rows = [&](int s0, int t0, int cnt) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = min(t0 + u, cnt - 1);
      const float* pa = pacc + (base + (size_t)(s0 + t) * g) * D + lane;
#pragma unroll
      for (int e = 0; e < E; ++e) part[u][e] = pa[64 * e];
    }
  };
  auto load_ml = [&](int s) {
    return s < n ? *reinterpret_cast<const float2*>(pml + (base + (size_t)s * g) * 2) : make_float2(-INFINITY, 0.f);
  };
  // The first 64 splits' (max, denominator) pairs, the first eight partial rows and the output
  // row's request metadata are all in flight together: a request of up to eight splits costs one
  // memory round trip before its arithmetic.
  float2 ml = load_ml(lane);
  if (n > 0) load_rows(0, 0, min(64, n));  // every decode request has at least one split
  const int4 m = w.meta[dr.x];
  float M = ml.x;
  for (int s = lane + 64; s < n; s += 64) M = fmaxf(M, pml[(base + (size_t)s * g) * 2]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  float den = 0.f, num[E];
#pragma unroll
  for (int e = 0; e < E; ++e) num[e] = 0.f;
  for (int s0 = 0; s0 < n; s0 += 64) {
    const int s = s0 + lane;
    if (s0 > 0) ml = load_ml(s);
    const float wgt = s < n ? fast_exp2(ml.x - M) : 0.f;
    den += s < n ? wgt * ml.y : 0.f;
    const int cnt = min(64, n - s0);
    for (int t0 = 0; t0 < cnt; t0 += 8) {
      if (s0 > 0 || t0 > 0) load_rows(s0, t0, cnt);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float wt = t0 + u < cnt ? __shfl(wgt, t0 + u) : 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) num[e] += wt * part[u][e];
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) den += __shfl_xor(den, off);
  const float inv = 1.0f / den;
  OutT* o = reinterpret_cast<OutT*>(out) + ((size_t)m.y * a.h_q + h) * D;
#pragma unroll
  for (int e = 0; e < E; ++e) o[lane + 64 * e] = static_cast<OutT>(num[e] * inv);
}

// Persistent: the grid holds as many waves as fit on the CUs the stream may use; each wave takes
// one item by its index, then the next ones from a counter until the list is exhausted (every
// wave reaches the exit).  Items are listed longest first.  Which wave computes an item never changes its arithmetic.
//
// A wave streams pages through a ring of kRing register buffers without a break at item
// boundaries: while it works on one item it takes the next one from the counter, reads the
// item's descriptor, then its page ids and query; the next item's first pages are loaded while
// the current item's last pages are computed.  Each item is processed in groups of kRing pages
// (the last group padded with masked pages that re-read the item's last page), so a page's
// buffer is known at compile time and a load is never separated from its use by an early exit.
// Per-wave LDS staging of finished items' partials (floats): up to kStageFloats / (g d + 2 g)
// items (7 for g = 4, d = 128) are written out together, when the buffer is full or the wave's
// work is done.  A store's completion comes back late while the memory system streams reads, and
// vector memory operations complete in order, so every store burst stalls the page loads issued
// after it until it completes: one burst per buffer instead of one per item.
//
// stage: this wave's buffer of kStageFloats floats in LDS.  Waves 0 .. n_waves - 1 start with the item
// of their index; a wave past them takes its first item from a counter as well.
constexpr int kStageFloats = 4096;
template <int D, int PPS>
__device__ __forceinline__ void decode_stream(const AttnArgs& a, const WorkArgs& w, float* const stage, int first,
                                              int n_waves) {
  constexpr int R = kRing;
  static_assert(PPS % R == 0, "a split must hold whole groups of ring pages");
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, quad = lane >> 4;
  const int g = a.group;
  const int n_items = w.n_ditems;
  const char* kcache = reinterpret_cast<const char*>(a.k_cache);
  const char* vcache = reinterpret_cast<const char*>(a.v_cache);
  // Both caches are [P, h_kv, 16 * d] in bytes per (page, head) slab; fold h_kv into the page stride.
  const long long slab_stride_pages = a.h_kv;

  const int ml_floats = (2 * g + 3) & ~3;
  const int item_floats = g * D + ml_floats;  // [g][d] output, then (m, l) per head
  const int n_slots = kStageFloats / item_floats;
  int n_staged = 0;     // items in the buffer
  int staged_rows = 0;  // lane k: partial row of buffered item k
  // Writes the buffered items to their partial rows, coalesced (LDS operations of one wave complete
  // in order, so the reads see the staging writes).
  auto flush = [&]() {
    for (int k = 0; k < n_staged; ++k) {
      const int row = __builtin_amdgcn_readlane(staged_rows, k);
      const float* src = stage + k * item_floats;
      float* dst = w.pacc + (size_t)row * g * D;
      for (int i = 4 * lane; i < g * D; i += 256)
        *reinterpret_cast<f32x4*>(dst + i) = *reinterpret_cast<const f32x4*>(src + i);
      if (lane < 2 * g) w.pml[(size_t)row * 2 * g + lane] = src[g * D + lane];
    }
    n_staged = 0;
  };

  // Wave v of the grid starts with item v; every item past the first n_waves is dealt round-robin
  // to n_queues counters (one atomic per item on a single counter would saturate it), and wave v
  // takes them from counter v % n_queues: ticket t is item n_waves + t n_queues + c.  Only one
  // item per wave is static, so from its second item on a wave that streams more slowly takes
  // fewer.  Every queue has a wave (n_waves >= n_queues), and a wave's tickets rise, as do their
  // items, all of them above the static ones: when a wave stops at an item past the end, every
  // ticket it still holds is past the end too.
  const int n_queues = n_waves >= kDecodeQueues ? kDecodeQueues : 1;
  const int queue = first % n_queues;
  int* const counter = w.work_counter + queue * kDecodeQueueStride;
  // The counter's old value, in lane 0; nothing touches it in the branch, so the load is waited
  // for only where it is read.
  auto grab = [&]() {
    int ticket = 0;
    if (lane == 0) ticket = atomicAdd(counter, 1);
    return ticket;
  };
  // An item's descriptor through the vector memory path, one word per lane: it completes in order
  // with the page loads issued before it, so waiting for it never drains the page stream.
  auto load_desc = [&](int idx) {
    return reinterpret_cast<const int*>(w.ditems)[(size_t)min(idx, n_items - 1) * 4 + (lane & 3)];
  };
  auto desc_item = [&](int words, int idx) {
    i32x4 v;
    v.x = __builtin_amdgcn_readlane(words, 0);
    v.y = __builtin_amdgcn_readlane(words, 1);
    v.z = __builtin_amdgcn_readlane(words, 2);
    v.w = __builtin_amdgcn_readlane(words, 3);
    return unpack_item(v, idx < n_items);
  };
  auto pages_of = [&](const DItem& it) { return min(PPS, (it.n_tok + 15) >> 4); };
  // The item's page ids, one per lane (at most PPS <= 64), and Q^T as the MFMA B operand:
  // column = head of the group, k = dims 32 ks + 8 quad .. +8.
  auto fetch_lane_data = [&](const DItem& it, int& ids, bf16x8 (&qf)[D / 32]) {
    const int* prow = a.page_table + (size_t)it.req * a.max_pages + it.first_page;
    ids = lane < pages_of(it) ? prow[lane] : 0;
    const __bf16* qrow = reinterpret_cast<const __bf16*>(a.q) + ((size_t)it.q_start * a.h_q + it.j * g + col) * D + quad * 8;
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) {
      const uint4 u = col < g ? *reinterpret_cast<const uint4*>(qrow + ks * 32) : make_uint4(0, 0, 0, 0);
      qf[ks] = __builtin_bit_cast(bf16x8, u);
    }
  };
  struct Ids {
    size_t slab;
    bool ok;
  };
  int bad = 0;
  // Page p (clamped to the item's last page) of an item whose ids a lane-distributed register holds.
  auto page_id = [&](int id_reg, int p, int n_pages, int j) {
    Ids r;
    const int id = __builtin_amdgcn_readlane(id_reg, min(p, n_pages - 1));
    r.ok = page_ok(id, a.num_phys_pages);
    bad |= !r.ok;
    r.slab = (size_t)(r.ok ? id : 0) * slab_stride_pages + j;
    return r;
  };

  // The deferred merge of the layer before: once a wave's item queue is empty (the launch's
  // tail, where waves would otherwise idle until the last items finish), it takes (request,
  // query head) pairs from merge queue `queue`: ticket t is pair t n_queues + queue.  Every queue
  // has a wave and every wave ends here, so every pair is merged.
  auto merge_tail = [&]() {
    if (w.n_merge == 0) return;
    int* const mcounter = w.work_counter + (kDecodeQueues + queue) * kDecodeQueueStride;
    for (;;) {
      int t = 0;
      if (lane == 0) t = atomicAdd(mcounter, 1);
      const int pair = __builtin_amdgcn_readfirstlane(t) * n_queues + queue;
      if (pair >= w.n_merge) break;
      merge_pair<D, __bf16>(a, w, w.merge_pacc, w.merge_pml, w.merge_out, pair, lane);
    }
  };
  if (first >= n_waves) first = n_waves + __builtin_amdgcn_readfirstlane(grab()) * n_queues + queue;
  if (first >= n_items) {
    merge_tail();
    return;
  }
  DItem cur = unpack_item(sload4(w.ditems + first), true);
  // The second item's ticket: its atomic returns while the first item's data loads.
  DItem nxt;
  {
    const int idx = n_waves + __builtin_amdgcn_readfirstlane(grab()) * n_queues + queue;
    nxt = desc_item(load_desc(idx), idx);
  }
  int cur_ids;
  bf16x8 qf[D / 32];
  fetch_lane_data(cur, cur_ids, qf);

  Page<D> buf[R];
  Ids ids[R];
  {
    const int np = pages_of(cur);
#pragma unroll
    for (int k = 0; k < R - 1; ++k) {
      ids[k] = page_id(cur_ids, k, np, cur.j);
      load_page<D>(buf[k], kcache, vcache, ids[k].slab, lane);
    }
  }

  for (;;) {
    const int n_pages = pages_of(cur);
    // At least two groups, so the next item's descriptor and ids (fetched in the first group)
    // are in before the last group loads its first pages.
    const int n_groups = max(2, (n_pages + R - 1) / R);
    const int n_tok = cur.n_tok;  // the item's tokens, from its first page on

    int ticket = 0, nn_words = 0, nn_idx = n_items, nxt_ids = 0;
    bf16x8 qn[D / 32];

    f32x4 acc[D / 16];
#pragma unroll
    for (int n = 0; n < D / 16; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    float l_run = 0.f;
    float m_ref = -INFINITY;  // reference max (base-2 units) the probabilities are taken against

    auto compute = [&](const Page<D>& pg, int p, const Ids& pid) {
      // Scores S^T: lane holds head `col`, tokens 4 quad + i of the page.
      f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks)
        sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pg.k[ks]), qf[ks], sc, 0, 0, 0);
      const int t0 = 16 * p + 4 * quad;
      // Tokens past the end (NaN-poisoned slots, and the padding pages of the last group) and
      // tokens of a bad page are masked; only the last pages of an item or a bad page need it.
      const bool tail = 16 * (p + 1) > n_tok || !pid.ok;
      if (tail) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (!pid.ok || t0 + i >= n_tok) sc[i] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
      mx = max_rows(mx);
      mx *= a.scale_log2;  // the scale is positive: max of scaled = scaled max
      // The reference max moves only when a score exceeds it by more than the slack, so the
      // output rescale is rare; numerator and denominator share the reference.
      if (__any(mx > m_ref + kRescaleSlack)) {
        const float m_new = fmaxf(m_ref, mx);
        const float alpha = fast_exp2(m_ref - m_new);
        m_ref = m_new;
        l_run *= alpha;
#pragma unroll
        for (int n = 0; n < D / 16; ++n) acc[n] *= alpha;
      }
      bf16x4 pb4;
#pragma unroll
      for (int i = 0; i < 4; ++i) pb4[i] = static_cast<__bf16>(fast_exp2(__builtin_fmaf(sc[i], a.scale_log2, -m_ref)));
      // The denominator sums the bf16 probabilities the PV product consumes.
      const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
      l_run = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pb4[0], pb4[1]}, ones, l_run, false);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pb4[2], pb4[3]}, ones, l_run, false);
      const s16x4 pbs = __builtin_bit_cast(s16x4, pb4);
      // Their values must not reach the MFMA either (0 x NaN is NaN).
      const uint64_t mk = !pid.ok ? 0ull : (tail ? low_elems_mask(n_tok - t0) : ~0ull);
#pragma unroll
      for (int n = 0; n < D / 16; ++n) {
        const uint64_t v = ((uint64_t)pg.v[n].y << 32 | pg.v[n].x) & mk;
        acc[n] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, v), pbs, acc[n], 0, 0, 0);
      }
    };

    // One group of R pages.  Every group issues the same loads in the same order (sources are
    // selected, never branched on), so the wait counts stay exact across the loop.  Items move
    // through a pipeline two deep: the first group takes a ticket for the item after next and
    // fetches the next item's ids and query; the last group reads the ticket (its atomic has
    // returned while the pages loaded after it did), loads that item's descriptor, then the next
    // item's first R - 1 pages (or, with no next item, re-reads).  No result is used right after
    // its load.
    auto group = [&](int grp, auto first_tag, auto last_tag) {
      constexpr bool kFirst = decltype(first_tag)::value;
      constexpr bool kLast = decltype(last_tag)::value;
#pragma unroll
      for (int u = 0; u < R; ++u) {
        if constexpr (kFirst) {
          if (u == 0) ticket = grab();
          if (u == 2) fetch_lane_data(nxt, nxt_ids, qn);  // a valid address even without a next item
        }
        if constexpr (kLast) {
          if (u == 0) {
            nn_idx = n_waves + __builtin_amdgcn_readfirstlane(ticket) * n_queues + queue;
            nn_words = load_desc(nn_idx);
          }
        }
        const int p = grp * R + u;
        const bool from_nxt = kLast && u > 0 && nxt.valid;
        const int src_ids = from_nxt ? nxt_ids : cur_ids;
        const int src_page = from_nxt ? u - 1 : p + R - 1;
        const int src_pages = from_nxt ? pages_of(nxt) : n_pages;
        const int src_j = from_nxt ? nxt.j : cur.j;
        ids[(u + R - 1) % R] = page_id(src_ids, src_page, src_pages, src_j);
        load_page<D>(buf[(u + R - 1) % R], kcache, vcache, ids[(u + R - 1) % R].slab, lane);
        compute(buf[u], p, ids[u]);
      }
    };
    using T = std::true_type;
    using F = std::false_type;
    group(0, T{}, F{});
    for (int grp = 1; grp < n_groups - 1; ++grp) group(grp, F{}, F{});
    group(n_groups - 1, F{}, T{});

    const float l_tot = sum_rows(l_run);
    {
      float* st = stage + n_staged * item_floats;
      if (col < g) {
#pragma unroll
        for (int n = 0; n < D / 16; ++n) *reinterpret_cast<f32x4*>(st + col * D + 16 * n + 4 * quad) = acc[n];
        if (quad == 0) {
          st[g * D + 2 * col + 0] = m_ref;
          st[g * D + 2 * col + 1] = l_tot;
        }
      }
      staged_rows = lane == n_staged ? cur.slot : staged_rows;
      ++n_staged;
    }
    if (n_staged == n_slots || !nxt.valid) flush();
    if (!nxt.valid) break;
    cur = nxt;
    nxt = desc_item(nn_words, nn_idx);
    cur_ids = nxt_ids;
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) qf[ks] = qn[ks];
  }
  if (bad && lane == 0) atomicOr(w.err, 1);
  merge_tail();
}

// Few items: one workgroup of 8 waves per item, each wave up to kSmallPages pages, all of their keys
// in flight at once.  A lone wave streams an item's 256 KiB in about 25 us whatever the rest of the
// chip does, since only three pages of it are in flight; eight waves with four pages each have
// the whole item in flight, and the time is one descriptor, one page-id and one page latency, then
// a merge of the waves through LDS.  Four requests of 620 .. 2783 tokens
// (32 / 8 heads of 128): 26.7 us before, 10.8 us now.  Short items of a long list share a workgroup
// (kernels.h, kSmallPair).
constexpr int kSmallWaves = 8;
constexpr int kSmallThreads = 64 * kSmallWaves;
constexpr int kSmallPages = kDecodePagesPerSplit / kSmallWaves;
static_assert(kSmallPages * kSmallWaves == kDecodePagesPerSplit, "the waves cover a split");
static_assert(kSmallPages % 2 == 0, "values are consumed two pages at a time");

// LDS of one workgroup: per wave its item's [g][D + 4] output and [g][2] (m, l), and the descriptors of
// its items; at most 68.7 KB (16 heads of 128).
constexpr int kSmallMaxPack = 4;  // items of a workgroup
template <int D>
constexpr size_t small_lds_bytes(int g) {
  return (size_t)kSmallWaves * g * (D + 4 + 2) * sizeof(float) + kSmallMaxPack * sizeof(int4);
}

// Workgroup `block` of small_blocks(w).  kPack: some of the items share a workgroup.
template <int D, bool kPack>
__device__ __forceinline__ void decode_items(const AttnArgs& a, const WorkArgs& w, int block, float* const lds) {
  constexpr int P = kSmallPages;
  constexpr int kStride = D + 4;  // floats per head in LDS: heads start on different banks
  const int tid = threadIdx.x;
  const int wave = uniform(tid >> 6);
  const int lane = tid & 63;
  const int col = lane & 15, quad = lane >> 4;
  const int g = a.group;
  // The workgroup's items first .. end - 1, W waves each.
  int W = kSmallWaves, first = block, end = block + 1;
  if (kPack && block >= w.n_small8) {
    const int blocks4 = (w.n_small4 + 1) / 2;
    if (block < w.n_small8 + blocks4) {
      W = 4;
      first = w.n_small8 + 2 * (block - w.n_small8);
      end = min(first + 2, w.n_small8 + w.n_small4);
    } else {
      W = 2;
      first = w.n_small8 + w.n_small4 + 4 * (block - w.n_small8 - blocks4);
      end = min(first + 4, w.n_ditems);
    }
  }
  const int sub = wave / W, wv = wave % W;  // the wave's item and its index among that item's waves
  const bool has = first + sub < end;
  const i32x4 desc = sload4(w.ditems + min(first + sub, end - 1));
  const DItem it = unpack_item(desc, has);
  const int n_tok = has ? it.n_tok : 0;  // a wave without an item: no page, no token
  const int n_pages = (n_tok + 15) >> 4;

  // Pages wv, wv + W, ... of the item.
  const int* prow = a.page_table + (size_t)it.req * a.max_pages + it.first_page;
  const int mine = lane < P && wv + W * lane < n_pages ? prow[wv + W * lane] : 0;
  bf16x8 qf[D / 32];
  const __bf16* qrow = reinterpret_cast<const __bf16*>(a.q) + ((size_t)it.q_start * a.h_q + it.j * g + col) * D + quad * 8;
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    const uint4 u = col < g ? *reinterpret_cast<const uint4*>(qrow + ks * 32) : make_uint4(0, 0, 0, 0);
    qf[ks] = __builtin_bit_cast(bf16x8, u);
  }
  // Every key page and the first half of the value pages load at once; the other half follows the
  // scores, so the wave fits in 128 registers and two workgroups in a CU.
  Page<D> pg[P];
  bool ok[P], bad = false;
  size_t slab[P];
  auto values = [&](int u) {
    if (ok[u]) {
      load_v<D>(pg[u], reinterpret_cast<const char*>(a.v_cache), slab[u], lane);
    } else {
#pragma unroll
      for (int n = 0; n < D / 16; ++n) pg[u].v[n] = make_uint2(0, 0);
    }
  };
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const int id = __builtin_amdgcn_readlane(mine, u);
    const bool there = wv + W * u < n_pages;
    ok[u] = there && page_ok(id, a.num_phys_pages);
    bad |= there && !ok[u];
    slab[u] = (size_t)(ok[u] ? id : 0) * a.h_kv + it.j;
    if (ok[u]) {
      load_k<D>(pg[u], reinterpret_cast<const char*>(a.k_cache), slab[u], lane);
    } else {
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) pg[u].k[ks] = make_uint4(0, 0, 0, 0);
    }
  }
#pragma unroll
  for (int u = 0; u < P / 2; ++u) values(u);
  f32x4 sc[P];
#pragma unroll
  for (int u = 0; u < P; ++u) {
    sc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks)
      sc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pg[u].k[ks]), qf[ks], sc[u], 0, 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = P / 2; u < P; ++u) values(u);
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < P; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (!ok[u] || 16 * (wv + W * u) + 4 * quad + i >= n_tok) sc[u][i] = -INFINITY;
      mx = fmaxf(mx, sc[u][i]);
    }
  const float m = max_rows(mx) * a.scale_log2;
  const float m_sub = m == -INFINITY ? 0.f : m;  // a wave without tokens: every weight is 2^-inf = 0
  bf16x4 pb[P];
  float l = 0.f;
  const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
#pragma unroll
  for (int u = 0; u < P; ++u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) pb[u][i] = static_cast<__bf16>(fast_exp2(__builtin_fmaf(sc[u][i], a.scale_log2, -m_sub)));
    // The denominator sums the bf16 probabilities the PV product consumes.
    l = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pb[u][0], pb[u][1]}, ones, l, false);
    l = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pb[u][2], pb[u][3]}, ones, l, false);
  }
  l = sum_rows(l);
  // Values two pages at a time: the contraction slots 0 .. 3 of a lane are the first page's
  // tokens 4 quad .. + 3, slots 4 .. 7 the second page's, in both operands.
  f32x4 acc[D / 16];
#pragma unroll
  for (int n = 0; n < D / 16; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < P; u += 2) {
    uint64_t mk[2];
#pragma unroll
    for (int x = 0; x < 2; ++x)  // values past the end must not reach the MFMA (0 x NaN is NaN)
      mk[x] = low_elems_mask(n_tok - (16 * (wv + W * (u + x)) + 4 * quad));
    const bf16x8 pf = {pb[u][0], pb[u][1], pb[u][2], pb[u][3], pb[u + 1][0], pb[u + 1][1], pb[u + 1][2], pb[u + 1][3]};
#pragma unroll
    for (int n = 0; n < D / 16; ++n) {
      const uint64_t v0 = ((uint64_t)pg[u].v[n].y << 32 | pg[u].v[n].x) & mk[0];
      const uint64_t v1 = ((uint64_t)pg[u + 1].v[n].y << 32 | pg[u + 1].v[n].x) & mk[1];
      const uint4 vf = make_uint4((unsigned)v0, (unsigned)(v0 >> 32), (unsigned)v1, (unsigned)(v1 >> 32));
      acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), pf, acc[n], 0, 0, 0);
    }
  }
  if (bad && lane == 0) atomicOr(w.err, 1);

  float* const ml = lds + kSmallWaves * g * kStride;  // [wave][g][2]
  i32x4* const descs = reinterpret_cast<i32x4*>(ml + kSmallWaves * g * 2);
  if (kPack && wv == 0 && lane == 0) descs[sub] = desc;
  if (col < g) {
    float* st = lds + (wave * g + col) * kStride;
#pragma unroll
    for (int n = 0; n < D / 16; ++n) *reinterpret_cast<f32x4*>(st + 16 * n + 4 * quad) = acc[n];
    if (quad == 0) *reinterpret_cast<float2*>(ml + (wave * g + col) * 2) = make_float2(m, l);
  }
  __syncthreads();
  // An item's waves in order, against their common max, one thread per four dims: the item's partial,
  // or the output itself where no request has a second split (there is no reduce kernel then).
  for (int x = tid; x < (end - first) * g * D / 4; x += kSmallThreads) {
    const int row = x / (D / 4), e = 4 * (x % (D / 4));
    const int s = kPack ? row / g : 0, c = row - s * g;
    const DItem t = kPack ? unpack_item(descs[s], true) : it;
    const float* const ml_s = ml + (s * W * g + c) * 2;
    const float* const acc_s = lds + (s * W * g + c) * kStride + e;
    float mm = -INFINITY;
#pragma unroll
    for (int v = 0; v < kSmallWaves; ++v)
      if (v < W) mm = fmaxf(mm, ml_s[v * g * 2]);
    const float mm_sub = mm == -INFINITY ? 0.f : mm;
    float den = 0.f;
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < kSmallWaves; ++v) {
      if (v >= W) break;
      const float2 p = *reinterpret_cast<const float2*>(ml_s + v * g * 2);
      const float wgt = fast_exp2(p.x - mm_sub);
      den += wgt * p.y;
      num += wgt * *reinterpret_cast<const f32x4*>(acc_s + (size_t)v * g * kStride);
    }
    if (w.max_split == 1) {
      const float inv = 1.0f / den;
      bf16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = static_cast<__bf16>(num[i] * inv);
      *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(a.out) + ((size_t)t.q_start * a.h_q + t.j * g + c) * D + e) = o;
    } else {
      *reinterpret_cast<f32x4*>(w.pacc + ((size_t)t.slot * g + c) * D + e) = num;
      if (e == 0) *reinterpret_cast<float2*>(w.pml + ((size_t)t.slot * g + c) * 2) = make_float2(mm, den);
    }
  }
}

// Clears the counter set of the partial kernel before this one on the stream (it has finished).
__device__ __forceinline__ void clear_previous_counters(const WorkArgs& w) {
  if (w.clear_counter && threadIdx.x < kDecodeSetLines) w.clear_counter[threadIdx.x * kDecodeQueueStride] = 0;
}

}  // namespace decode
}  // namespace duet
