// Launch interface between the runtime and the HIP kernels (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "duet.h"

namespace duet {

// Per-iteration tensors and shape, common to every attention kernel.
struct AttnArgs {
  const void* q;         // [T, h_q, d]
  const void* k_cache;   // [P, h_kv, 16, d]
  const void* v_cache;   // [P, h_kv, d, 16]
  const int32_t* page_table;
  void* out;             // [T, h_q, d]
  long long num_phys_pages;
  int32_t max_pages;     // row stride of page_table
  int32_t h_q, h_kv, group, head_dim, dtype;
  float scale_log2;      // log2(e) / sqrt(d): scores are kept in base-2 units
};

// One prefill workgroup's work: query rows row0 .. of a request for some heads from `head` on (bf16: all
// heads of the unit; fp32: one), over key tiles [tiles & 0xffff, tiles >> 16).  Everything a
// workgroup needs to start, in one read.
struct PrefillItem {
  int32_t req, head, row0;
  int32_t slot;  // -1: a whole unit, else piece_slot of a piece
  int32_t q_start, q_len, cached_len;
  uint32_t tiles;
};
// A piece's slot; for a unit that merges itself also the piece's index in it (its pieces have
// consecutive slots) and the number of pieces (0: the merge kernel merges them).
inline int32_t piece_slot(int slot, int piece, int pieces_to_merge) { return slot | piece << 16 | pieces_to_merge << 24; }
// A prefill unit whose pieces the merge kernel merges: slots slot .. slot + pieces - 1.
struct PrefillUnit {
  int32_t slot, pieces;
  int32_t req, head, row0, q_start, q_len, pad;
};

// Work lists and scratch that live in the caller's workspace.
struct WorkArgs {
  const int4* meta;     // [R]  (kind, q_start, q_len, cached_len)
  const PrefillItem* pitems;  // [NP] heaviest first
  const int4* dreq;     // [RD] decode requests (req, item_base, n_split, n_pages)
  float* pacc;          // [ND, group, d]  unnormalised split-K partial outputs
  float* pml;           // [ND, group, 2]  (running max in base-2 units, softmax denominator)
  const int4* ditems;   // [ND] bf16 decode items in execution order: (q_start, req | kv head << 24,
                        //      first page | (tokens - 1) << 22, row of the item's partial)
  int32_t* err;         // error word: bit 0 = page id out of range
  int32_t* work_counter;  // kDecodeSetInts ints: this launch's counter set (see kDecodeQueues)
  int32_t* clear_counter; // counter set a bf16 partial kernel clears when it starts, or null
  // Deferred merge (bf16): the split-K partials of the layer before, merged by this partial
  // kernel's waves once its item queue is empty.  n_merge = 0: nothing to merge.
  const float* merge_pacc;
  const float* merge_pml;
  void* merge_out;        // that layer's output
  int32_t n_merge;        // (decode request, query head) pairs
  int32_t n_pitems, n_dreq, max_split, n_ditems;
  int32_t decode_pps;     // pages per bf16 decode item
  int32_t decode_small;   // bf16 decode items run one workgroup each and merge themselves (decode_rule)
  int32_t n_small8, n_small4;  // of those items, longest first: run with 8 waves, with 4; the rest with 2
  int32_t decode_cus;   // CUs the decode stream may use (sizes the persistent grid)
  int32_t prefill_cus;  // CUs the prefill stream may use
  int32_t prefill_id_cap;  // most pages of any prefill request (sizes the LDS page-id table)
  // Prefill key split (bf16, see kPrefillPieceFill).
  float* ppart;               // [slots] partial state of every piece: unnormalised O, running max, denominator
  int32_t* pcount;            // [slots] pieces finished, at the unit's first slot; zero before and after every launch
  const PrefillUnit* punits;  // [n_punits] units for the merge kernel
  int32_t n_punits;
  long long prefill_tiles;      // key tiles over all units (bf16)
  int32_t prefill_longest;      // key tiles of the longest item (bf16)
};

inline int small_blocks(const WorkArgs& w) {
  return w.n_small8 + (w.n_small4 + 1) / 2 + (w.n_ditems - w.n_small8 - w.n_small4 + 3) / 4;
}

// Cache writes of look-ahead decode steps: new key and value rows in, paged cache out.  Job x writes step
// x / layers + 1 of layer x % layers.
struct AppendJob {
  const void* k_new;     // [R_d, h_kv, d], decode requests in order
  const void* v_new;     // [R_d, h_kv, d]
  void* k_cache;         // [P, h_kv, 16, d], written
  void* v_cache;         // [P, h_kv, d, 16], written
};
struct AppendArgs {
  const AppendJob* jobs;
  const int32_t* page_table;
  long long num_phys_pages;
  int32_t max_pages;
  int32_t h_kv, head_dim, dtype;
  int32_t first_job, n_jobs, layers;  // jobs first_job .. first_job + n_jobs - 1
};

// Decode split length in pages.
constexpr int kDecodePagesPerSplit = 32;  // bf16, most batches
constexpr int kDecodePagesPerSplitF32 = 2;
// Most logical pages of a bf16 decode request (an item's first page is a 22-bit field).
constexpr long long kMaxDecodePages = (1LL << 22) - 1;

// The persistent decode kernel's work queue is split into kDecodeQueues counters (items are dealt
// round-robin to them), each on its own 128-byte line: atomics on one line are serialised, at a
// few tens per microsecond.  A counter set is kDecodeQueues item queues followed by kDecodeQueues
// merge queues (the deferred merge of the layer before).  A call has two sets, which consecutive
// layers alternate: the upload zeroes both, a partial kernel clears the set the kernel before it
// on the stream used (that kernel has finished), and a reduce kernel clears the set of the
// partial kernel it follows.
constexpr int kDecodeQueues = 8;
constexpr int kDecodeQueueStride = 32;  // ints: one 128-byte line per counter
constexpr int kDecodeSetLines = 2 * kDecodeQueues;
constexpr int kDecodeSetInts = kDecodeSetLines * kDecodeQueueStride;
constexpr int kDecodeCounterInts = 2 * kDecodeSetInts;

// How a batch's bf16 decode work is cut, from its items at kDecodePagesPerSplit pages per item and
// the most pages of a request.  The rule depends on the batch only, so results are the same for
// every CU split; where two cuts trade the shares against each other, it takes the one that loses on
// none of them by more than a few per cent.  Decode time of one layer (us), 32 / 8 heads of 128,
// on 256, 128 and 32 CUs:
//   one split per request: a workgroup per item wins (contexts of 300 tokens, 64 items
//     8.8 / 17 / 17 against 20.6 / 24 / 24 streamed; 512 items 18.8 / 29 / 79 against
//     26.7 / 34 / 91; 4096 items 117 / 175 / 565 against 146 / 203 / 670), if short items share
//     one (below);
//   few items: a workgroup per item (contexts of 2048, 64 items 13.4 / 19.0 / 23.5 against
//     28.0 / 31.5 / 31.5; from 128 items on 32 CUs lose, 37.4 against 34.3);
//   then half as long items, streamed (128 items 18.6 / 22.2 / 34.6 against 29.1 / 32.9 / 34.3; 256
//     items 21.5 / 25.2 / 59.7 against 30.7 / 34.8 / 59.1; 384 items still gain on 256 CUs, 26.3
//     against 33.0, but lose 2-4% on 32).
constexpr int kDecodePagesPerSplitShort = 16;
constexpr int kSmallMaxItems = 96;
constexpr int kShortMaxItems = 256;
// A workgroup's eight waves take four pages each, so a short item alone leaves most of them without one,
// which costs nothing while every CU has at most one item and a lot on small shares of long lists.  From
// kSmallPair items on those of at most 16 pages run two to a workgroup, from kSmallQuad on those of at
// most 8 pages four (fewer, and the whole chip would idle).  One layer of 16 (us), 16 / 8 heads of 128,
// on 256, 96 and 32 CUs, streamed, a workgroup each, shared: contexts of 100 to 127, 512 items
// 14.7 / 22.2 / 45, 10.8 / 24.2 / 54, 10.5 / 19 / 35; 1024 items 22 / 36 / 82, 19 / 40 / 101, 15 / 26 / 56;
// 4000 items 63 / 111 / 294, 60 / 133 / 371, 48 / 81 / 201; contexts of 60 to 200, 4000 items 67 / 121 / 324,
// 63 / 135 / 374, 52 / 85 / 218.  At 256 items sharing loses on the whole chip (contexts of 30 to 60
// 5.6 against 6.4) and a workgroup each on 32 CUs only a little against streaming (100 to 127: 27.5 against 26.4).
constexpr int kSmallPair = 257, kSmallQuad = 1024;
struct DecodeRule {
  int pages_per_split;
  bool small;  // decode_small_bf16: one workgroup per item, or per 2 or 4 short ones
  int n8, n4;  // of its items, longest first: run with 8 waves, with 4; the rest with 2
};
inline DecodeRule decode_rule(int64_t n_items, int max_pages) {
  if (max_pages <= kDecodePagesPerSplit || n_items <= kSmallMaxItems) return {kDecodePagesPerSplit, true, 0, 0};
  if (n_items <= kShortMaxItems) return {kDecodePagesPerSplitShort, false, 0, 0};
  return {kDecodePagesPerSplit, false, 0, 0};
}

// Keys a prefill request may attend (its page ids are staged in LDS: 8192 ids, 32 KB).
constexpr int kMaxPrefillKeys = 131072;

constexpr int kPrefillRows = 128;  // query rows per fp32 prefill item (8 workgroups x 16)
constexpr int kPrefillKeys = 64;   // keys per LDS stage (4 pages)

// bf16 prefill work unit: prefill_heads_per_unit(group) query heads of one GQA group times
// prefill_rows_per_unit(group, dtype) queries.  fp32 items are one head times kPrefillRows.
int prefill_heads_per_unit(int group);
int prefill_rows_per_unit(int group, int dtype);

// Prefill key split (bf16).  Let T be the batch's total key tiles (kPrefillKeys keys) over all
// units and P = max(kPrefillPieceMinTiles, ceil(T / kPrefillPieceFill)), an even share of the
// batch over one workgroup per CU of the whole chip.  A unit whose causal key range spans more
// than 1.5 P tiles runs as n = ceil(tiles / P) pieces of ceil(tiles / n) consecutive tiles (the
// last may be shorter; n is recounted so that none is empty), so a short chunk after a long
// cached prefix (few units, each long) still fills the CUs.  Every piece pays a fixed start-up
// cost and a partial-state round trip, so units within 1.5 P of the share stay whole.  P depends
// on the batch only, never on the CU split, so results are the same for every split.  Each piece
// writes its partial state to a slot.  Of up to kPrefillSelfMerge pieces the last to finish (a
// counter per unit) merges the slots in piece order and writes the output; the slots of more
// pieces are merged by a kernel of their own.  Split units number at most
// T / P <= kPrefillPieceFill and their slots at most 2 T / P, plus the tail split's below
// (kPrefillPieceFill units, kPrefillTailPieces slots each).
constexpr int kPrefillPieceMinTiles = 8;
constexpr int kPrefillPieceFill = 256;
// Tail split (batch-only as well): when the whole units number at least 2 kPrefillPieceFill, the
// kPrefillPieceFill shortest of them (dispatched last) run as kPrefillTailPieces pieces, each of
// at least kPrefillTailMinTiles tiles, so the last round of workgroups is fine-grained on any share
// (one workgroup per CU leaves up to one unit's length idle at the end otherwise).
constexpr int kPrefillTailPieces = 4;
constexpr int kPrefillTailMinTiles = 16;
// One workgroup reads a piece's 128 KiB in about 2 us, whatever the other CUs do; a kernel reads all of
// them on every CU but takes about 10 us with its launch.  One layer (us), merged by the last piece
// against by a kernel: two pieces (2048 tokens, 32 / 8 heads) 53.5 / 60.5; tail split in four (8192
// tokens) 513 / 529; five (8 / 1 heads, 1500 tokens after 900) 35.7 / 40.1; eight (4 / 4 heads, 2048
// after 2048) 42.4 / 33.2; 16 (32 / 8 heads, 16 tokens after 8000) 51.7 / 30.0; 33 (4 / 4 heads, 512
// after 16384) 88.6 / 44.5.
// Units of more than six beside units of fewer (us a layer, 1500 tokens after 2341, 8 / 1 heads, on 256 CUs;
// 872 after 2341, 8 / 2 heads, on 160): each by its last piece 42 / 50; the short ones so and the long ones
// by the kernel 48 / 57; all by the kernel 37 / 44.
constexpr int kPrefillSelfMerge = 6;
static_assert(kPrefillTailPieces <= kPrefillSelfMerge, "the tail split merges itself");
static_assert(2 * kPrefillPieceFill + kPrefillPieceFill * kPrefillTailPieces <= 0xffff, "a slot fits 16 bits");
static_assert(kMaxPrefillKeys / kPrefillKeys <= 0xffff, "a tile index fits 16 bits");
int prefill_piece_tiles_for(long long total_tiles);
size_t prefill_slot_bytes(int head_dim);  // one piece's partial state

// The QKV-split step of a block (bf16): query rows out, new keys and values into the cache.
struct QkvSplitArgs {
  const __bf16* qkv;       // [T, (h_q + 2 h_kv) d] projection output
  __bf16* q;               // [T, h_q, d]
  __bf16* k_cache;         // [P, h_kv, 16, d]
  __bf16* v_cache;         // [P, h_kv, d, 16]
  const int4* meta;        // [R] (kind, q_start, q_len, cached_len), q_start rising
  const int4* dreq;        // null: a row's request is found by q_start; else row i is decode request i
                           //       (dreq[i].x) of a look-ahead step
  const int32_t* page_table;
  long long num_phys_pages;
  int32_t* err;
  int32_t num_reqs, max_pages, h_q, h_kv, head_dim;
  int32_t row0, rows;      // the launch's rows
};

// Projections of few rows (gemm_skinny.hip) instead of the library's, for a partition of `rows` rows on
// `cus` CUs and layers of model width d, QKV width d_qkv and MLP width m: where one part of the widest product in
// fp32 fits in `bytes` (at 64 rows more than 131072 columns do not), and where they are faster.  A layer
// behind 130 us of attention (us gained over the library's kernels and the operators they fuse), whole chip / 128 /
// 96 / 64 / 32 CUs:
//   up to 32 rows they gain on the whole chip for every size (436 MB of weights, Llama-3-8B, 16 rows 78; 6 MB 2), and
//   from 96 CUs on up to 436 MB (16 rows: 436 MB 78 / 24 / 11; 50 MB 16 / 14 / 17); below that the weights a CU
//   pulls count, at about 30 GB/s (16 rows: 30 MB 15 / 17 / 17 / 17 / 17, 436 MB on 64 and 32 CUs -30 and -60; 32 rows:
//   30 MB on 32 CUs 9, 201 MB 23), and the host's share: a library call costs it about 20 us, which the own
//   kernels' fewer launches save where nothing else is slower, so sizes with little to gain keep to
//   rows times weights against the CUs;
//   past 32 rows the partial sums of products of d columns weigh as much as the weights: behind narrow MLPs, whose
//   gate-up has few workgroups too, they lose (64 rows, d 1536: m 512 -5 / -6 / . / -17, m 1584 2 / 1 / . / -20,
//   m 4096 10 / 3 / 4 / -7 / -57; d 2048: m 512 -3 / -12 / . / -32, m 4096 9 / -5 / -14 / -29 / -108); widths near 1024
//   gain on every share their weights suit (17 MB 9 / 10 / 9 / 10 / -2), and MLPs of twice d and more on the
//   whole chip (436 MB 78, d 2048 with m 6144 27).
// The two round their sums in different orders, so a block's result may differ in its last bits between
// shares on different sides of the rule.
constexpr int kSkinnyRows = 64;
bool use_skinny(int rows, int cus, int d, int d_qkv, int m, size_t bytes);
struct SkinnyArgs {
  const __bf16* x;  // [rows, d_in]
  const __bf16* w;  // [d_in, d_out]
  float* part;      // [splits, rows, d_out]
  __bf16 *gu, *act; // gate-up: [rows, 2 m], [rows, m]
  int32_t rows, d_in, d_out, m, splits, tiles;
};
// At least one, whether or not one part fits in `bytes` (use_skinny).
int skinny_splits(int rows, int d_in, int d_out, size_t bytes);
hipError_t launch_skinny_gemm(const __bf16* x, const __bf16* w, float* part, int rows, int d_in, int d_out, int splits,
                              hipStream_t s);
hipError_t launch_skinny_gate_up(const __bf16* x, const __bf16* w, __bf16* gu, __bf16* act, int rows, int d_in, int m,
                                 hipStream_t s);
hipError_t launch_residual_norm(const float* part, int splits, __bf16* x, const __bf16* w, __bf16* y, int rows, int d,
                                float eps, hipStream_t s);
hipError_t launch_qkv_finish(const float* part, int splits, __bf16* qkv, const QkvSplitArgs& a, hipStream_t s);

hipError_t launch_rmsnorm(const __bf16* x, const __bf16* w, __bf16* y, int rows, int d, float eps, hipStream_t s);
hipError_t launch_swiglu(const __bf16* gu, __bf16* a, int rows, int m, hipStream_t s);
hipError_t launch_qkv_split(const QkvSplitArgs& a, hipStream_t s);

hipError_t launch_decode_partial(const AttnArgs& a, const WorkArgs& w, hipStream_t s);
hipError_t launch_decode_reduce(const AttnArgs& a, const WorkArgs& w, hipStream_t s);
hipError_t launch_prefill(const AttnArgs& a, const WorkArgs& w, hipStream_t s);
// Merges the units that ran as pieces (bf16; launch_prefill and launch_mixed end with it).
hipError_t launch_prefill_merge(const AttnArgs& a, const WorkArgs& w, hipStream_t s);
// Both bf16 halves of a layer in one launch, where that gains: not when prefill lasts so much longer
// that decode hardly matters, nor for many small decode items, two of which fit on a CU that
// runs no prefill (us a layer, one launch against two: 512 new tokens beside 32 items 25 / 34,
// beside 1600 items 84 / 79; 64 tokens beside 800 items 33 / 32).  One launch against two, heads of 128, by
// key tiles per decode item: 59, 5% faster; 100 to 256, from 7% faster (8 / 1 heads, 4096 tokens after
// 16384 beside 64 decodes 372 / 399) to 1.4% slower (64 / 8 heads, 8192 after 8192 beside 64, 3043 / 3000),
// 1.4% faster on average; past 256, within 2.6% either way, but 8 / 1 heads still 1 to 7% faster.
// Heads of 64 keep the rule: one launch is 5 to 20% faster but where a long chunk's prefill alone runs
// two workgroups per CU (16 / 2 heads, 100 decodes: beside 8192 tokens 220 / 264, after 8192 557 / 542, after
// 24576 1191 / 1106), and where hardly any prefill is beside decode that lasts about three items a wave, whose
// waves sit on fewer CUs (2686 items beside 10 tokens 86 / 76, beside 512 96 / 100; 3406 beside 10 to 200
// tokens 111 to 116 / 95 to 100; but 1268 items beside 64 53 / 58, 7108 beside 200 0.98 of two): there two launches.
constexpr int kMixedMaxTilesPerItem = 256;
constexpr int kMixedMaxSmallItems = 512;
inline bool use_mixed(const AttnArgs& a, const WorkArgs& w) {
  if (w.n_ditems == 0 || w.n_pitems == 0 || (w.decode_small && w.n_ditems > kMixedMaxSmallItems)) return false;
  if (a.head_dim == 64 && !w.decode_small && w.n_ditems > 2048 && w.n_ditems <= 6144 && 16 * w.prefill_tiles < w.n_ditems)
    return false;
  return w.prefill_tiles <= (long long)kMixedMaxTilesPerItem * w.n_ditems;
}
hipError_t launch_mixed(const AttnArgs& a, const WorkArgs& w, hipStream_t s);
// The fp32 paths of the two launchers above.
hipError_t launch_decode_partial_f32(const AttnArgs& a, const WorkArgs& w, hipStream_t s);
hipError_t launch_prefill_f32(const AttnArgs& a, const WorkArgs& w, hipStream_t s);
// Writes the new tokens of every decode request in w.dreq (step 0's lists) for the launch's jobs.
hipError_t launch_kv_append(const AppendArgs& a, const WorkArgs& w, hipStream_t s);

hipError_t launch_gather(const void* cache, int which, int elem_bytes, int h_kv, int d, const int32_t* page_table,
                         int max_pages, long long num_phys, int req, int kv_len, void* out, int32_t* err,
                         hipStream_t s);

// Copies `bytes` (a multiple of 16, as zero_bytes) of host-visible memory to dst, the first zero_bytes
// of dst as zeros; workgroup b < upload_blocks(bytes) <= kUploadBlocks then writes seq to flags[b].
constexpr int kUploadBlocks = 64;
int upload_blocks(size_t bytes);
hipError_t launch_upload(const void* src, void* dst, size_t zero_bytes, size_t bytes, uint32_t* flags, uint32_t seq,
                         hipStream_t s);
// Copies `bytes` (a multiple of 4) of host memory to dst as kernel arguments: src may change as soon as
// the call returns, also where the launches are captured.
hipError_t launch_upload_by_value(const void* src, void* dst, size_t bytes, hipStream_t s);

hipError_t launch_read_probe(const void* buf, size_t bytes, int blocks, unsigned* sink, hipStream_t s);
size_t read_probe_bytes(size_t bytes, int blocks);
hipError_t launch_mfma_probe(int blocks, int iters, float* sink, hipStream_t s);
hipError_t launch_placement_probe(int blocks, uint32_t* out, hipStream_t s);

}  // namespace duet
