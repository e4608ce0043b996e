// Internal declarations shared by the translation units of libtt_emb.so (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "tt_emb.h"

namespace ttemb {

constexpr int kWave = 64;

// Stable counting-sort blocks: every wavefront owns 256 consecutive items of its block's run.
constexpr int kSortWaveItems = 256;
__host__ __device__ constexpr int sort_items(int threads) { return threads / kWave * kSortWaveItems; }
constexpr int kChunk3 = 16;       // record slots per partial sum (chunk) of a G3 slice gradient
// Batches of up to kSmallBatch rows are cut finer where that puts more wavefronts in flight: by-i3
// chunks of 8 ids instead of 16 (-3.7 us per step at 200,000 rows, +6..18 us at 500,000).
constexpr int kSmallBatch = 1 << 18;
constexpr int kChunk3Min = 8;
inline int chunk3_fill(int64_t B) { return B <= kSmallBatch ? kChunk3Min : kChunk3; }

// Threads of a sort block.  A block's time goes into what its wavefronts do between barriers, not
// into memory: on an idle device smaller blocks on more compute units are faster until the 2048
// counters per block outweigh them (training step, microseconds with 256 / 512 / 1024 threads:
// 50,000 ids 113 / - / 118, 100,000 items 126 / - / 139, 200,000 ids 194 / 192 / 197, 500,000 ids
// - / 404 / 408).  Up to kSort1024First items, one block of either kind, 1024 threads have an eighth of
// the counters each: a pass over 700 items 9.8 against 11.2 us (5,000 uniform ids are slower with them, a
// step 99 against 93).  Beside the arithmetic of another batch (tt_emb_prepare) the extra blocks take its
// compute units instead: 156 / 150 / 145 at 200,000 ids, so there they stay large.
constexpr int kSort1024First = 1 << 10, kSort256Most = 1 << 17, kSort512Most = 1 << 19;
inline int sort_threads(int64_t B, bool beside) {
  return beside || B <= kSort1024First || B > kSort512Most ? 1024 : B > kSort256Most ? 512 : 256;
}
inline int64_t sort_blocks(int64_t B) {
  const int i = sort_items(sort_threads(B, false));
  return (B + i - 1) / i;
}
// most blocks that any batch of up to maxB items is sorted by
inline int64_t sort_blocks_most(int64_t maxB) {
  int64_t m = sort_blocks(maxB);
  for (int64_t b : {(int64_t)kSort256Most, (int64_t)kSort512Most})
    if (b < maxB && sort_blocks(b) > m) m = sort_blocks(b);
  return m;
}
constexpr int kMaxBins = 2048;                            // digit / bucket count limit per pass

// The unit of the gradient sums: a run of equal ids is cut at every multiple of kEntrySlots sorted
// slots, and each piece ("entry") is carried through the backward pass like an id of its own - all
// gradient steps are linear in the row gradient, so the pieces of an id simply add up in the same
// matrix-core accumulations that add up the ids of a prefix or of an i3 group.  A block of the
// gradient-sum kernel owns kEntrySlots slots, so no sum ever crosses a block.  (Pieces of 256 shorten
// that kernel, 21 -> 18 us at 200,000 Zipf ids, but the hot prefix's pieces queue up behind each other in
// the next one, 50 -> 88.)
constexpr int kEntrySlots = 1024;

constexpr int kXcds = 8;
// walk_chunks3: most chunks of a column, in mean groups' eighths, and the chunks that a group has on average for each
// XCD where groups are walked at all (both sides measured there).
constexpr uint32_t kWalkMeans = 2;
constexpr int kWalkLeast = 2;

constexpr int kTileSlots = 32;   // sorted slots per wavefront tile in the row kernels
constexpr int kChunk2 = 16;      // unique prefixes per partial sum of a G2 slice gradient

// Where the ids of a batch come from, passed to the first sort pass by value.
struct IdSource {
  const int64_t* ids;      // device [B]; nullptr: the consecutive ids base, base+1, ...
  int64_t base;
  const int32_t* reindex;  // device [n_ids] old id -> table row, or nullptr (ids are table rows)
  int64_t n_ids;
  // Slab split (see Plan::split): item idx of the pipeline is slab idx % split of batch position
  // idx / split; rows is the caller's table size N and n23 = n2*n3.
  int split;
  int64_t rows, n23;
};
// The same for lookups by prefix (split is 1): the key is not the table row but
// (i2*n1 + i1) << i3_bits | i3, see Plan::lookup_keys.  A type of its own: with a branch on it in key_of_id,
// whose arguments and divisions k_direct_fwd then carries too, index-free calls took 1 to 4 % longer (2,048
// ids and fewer, 7 to 25 us).
struct PrefixSource {
  IdSource ids;
  int i3_bits;
  uint32_t n1, n2, n3;
};

// What a sort orders by: `bits` bits of the key above the lowest `low`, `per` of them a pass.
// Out-of-range ids have the key `sentinel`, above every other.  The first pass reads key buffer 1 (which
// its histogram fills from the ids) and writes the other, the next one back, and so on.
struct SortKeys {
  uint32_t sentinel;
  int low, bits, passes, per;
  int sorted() const { return (passes + 1) & 1; }  // buffer of the sorted keys
  int bits_of(int pass) const { return std::min(per, bits - pass * per); }
};

// Words of eight 16-bit counts in a row of a sort block.
__host__ __device__ constexpr int sort_row_words(int bins) { return bins < 8 ? 1 : bins / 8; }

// Whether the scatter blocks add up the histograms' columns themselves, or a column-scan launch does it: every
// block reads all rows, so the line lies at a number of 16-byte words of them.  Training steps, the launch
// against the sums: 49 blocks of 64 words 87.4 / 84.1 us, 98 of 128 104.4 / 103.7, beside another batch's
// arithmetic 49 of 256 121.1 / 122.8, 98 of 256 163.4 / 168.6 (and 245 of 64 even).
constexpr int kFoldWords = 8192;
inline bool sort_folds(const SortKeys& sk, int64_t B, int pass, bool beside) {
  const int items = sort_items(sort_threads(B, beside));
  return (B + items - 1) / items * sort_row_words(1 << sk.bits_of(pass)) <= kFoldWords;
}


// Update rule of the update kernel and its caller-owned state (arrays shaped like the cores).
enum UpdateKind { kUpdateSgd = 0, kUpdateAdagrad = 1, kUpdateAdam = 2 };
struct UpdateRule {
  int kind;
  float *s1, *s2, *s3;  // Adagrad: running sums of squared gradients; Adam: first moments
  float *v1, *v2, *v3;  // Adam: second moments
  float eps;
  float beta1, beta2;   // Adam decay rates
  float corr1, corr2;   // Adam bias corrections 1/(1 - beta1^t), 1/(1 - beta2^t) of this step
};

// Table and slice geometry, passed to kernels by value.
struct Shape {
  uint32_t n1, n2, n3, N;  // node factors and N = n1*n2*n3
  int d1, d2, d3, r1, r2;
  int M;   // d1*d2       rows of the partial product
  int W;   // d2*r2       columns of the unfolded G2 slice
  int PN;  // d1*d2*r2    floats of one prefix product
  int D;   // d1*d2*d3    floats of one embedding row
  int S1;  // d1*r1       floats of one G1 slice
  int S2;  // r1*d2*r2    floats of one G2 slice
  int S3;  // r2*d3       floats of one G3 slice
};

__host__ __device__ constexpr int up8(uint32_t n) { return (int)(n + 7) & ~7; }

// Sorted slots of a block of the segment and grouping kernels, a quarter of them threads of the latter: few, for many
// blocks, up to a block a compute unit and as long as a grouping block adds up the counts of all blocks, a row of
// 16-byte words of eight buckets each, in five rounds of eight rows a group of threads.  Beside another batch's
// arithmetic, which the loads of those rows disturb, up to a number of words in all.  Training steps in us with
// 1024 / 2048 / 4096 slots, uniform ids, rank 16, d = (4,4,4), n1 = 136, and the rows of 1024 slots and their words:
//   n2 = n3 = 136           100,000 ids, 98 x 17: 114 / 116 / 122       200,000, 196 x 17: 149 / 150 / 156
//                           400,000, 391 x 17: 221 / 218 / 223          600,000, 586 x 17: 299 / 298 / 293
//   n2 = 136, n3 = 480      150,000, 147 x 60: 138 / 140 / 145          250,000, 245 x 60: 176 / 173 / 178
//                           500,000, 489 x 60: - / 258 / 262            600,000, 586 x 60: - / 309 / 305
//   n2 = 100, n3 = 1000     90,000, 88 x 125: 118 / 118 / 124           150,000, 147 x 125: 141 / 140 / 146
// and beside, 100,000 Zipf ids of 480x480x482 at rank 64 (98 x 60) 451 / - / 470, 200,000 of 136^3 at rank 32
// (196 x 17) 124 / 123 / 124, 400,000 uniform ones of 100^3 (391 x 13) 170 / 172 / 174, 100,000 of 50x100x2000 at
// rank 32 (98 x 250) - / 109 / 106, 500,000 Zipf ids of 480x480x482 (489 x 60) 348 / 334 / 331, 800,000 510 / 479 / 472.
// The counts lie in the memory that Workspace::seg_rows names, which holds at least 8192 + 4*n3 bytes per 4096 slots.
constexpr int kSlotBlocks = 256, kSlotRounds = 5, kSlotWordsBeside = 8192;
inline int slot_span(const Shape& sh, int64_t B, bool beside) {
  const int p3 = up8(sh.n3), p2 = up8(sh.n2), words = std::max(p3, p2) / 8;
  int span = 1024;
  auto too_many = [&](int64_t blocks) {
    const int rows = std::max(span / 4 / words, 1) * 8;  // of a round
    return beside ? blocks * words > kSlotWordsBeside : blocks > kSlotBlocks || blocks > (int64_t)kSlotRounds * rows;
  };
  while (span < 4096 &&
         (too_many((B + span - 1) / span) || 4096 / span * 2 * (p3 + p2) > 8192 + 4 * (int)sh.n3))
    span *= 2;
  return span;
}

// Device-side counters of the latest forward (first bytes of the workspace).
struct Counters {
  int U;        // entries: distinct in-range ids, long runs counted once per kEntrySlots piece
  int Q;        // distinct (i1,i2) prefixes
  int nvalid;   // in-range batch positions (they occupy sorted slots [0, nvalid))
  int nchunk3;  // partial-sum chunks over the by-i3 grouping of unique ids
  int nchunk2;  // partial-sum chunks over the by-i2 grouping of unique prefixes
  int err;      // nonzero: a kernel met an impossible index (bit mask of sites)
  int n_split;  // entries beyond the first of their id (U - n_split distinct ids)
  int walk_cols, walk_steps;  // columns in walk3 (none: chunks in index order), chunks of one that an XCD takes
  int small;    // ranks 64 and 128: an operand of the prefix kernels is below 2^-102 and not zero
};

// Scratch of the index-free kernels for small batches (tt_emb_direct.hip), sized for
// Plan::direct_train_cap items (the keys for Plan::direct_cap; tt_emb_get_stats reads them).
struct DirectBuffers {
  uint32_t* key;    // item -> table row, or the sentinel N; kept for tt_emb_get_stats
  uint16_t* dig;    // [3][stride]: i1, i2, i3 of every item, 0xffff for an out-of-range id
  int stride;       // items per digit row, a multiple of 8
  float* P;         // prefix product of every item           [cap][PN]
  float* dP;        // gradient of that product               [cap][PN]
  float* g1;        // its G1 slice before the update         [cap][S1]
  float* dg1;       // its term of dG1[i1]                    [cap][S1]
  float* dg3;       // its term of dG3[i3]                    [cap][S3]
  // parts of slices that many items share (k_direct_apply), listed by the backward kernel
  int2* hot;        // {slice, part number from 1 on}       [3 cores][hot_parts]
  uint32_t* n_hot;  // parts listed per core; then tickets  [3] + [3*hot_parts][pieces of a slice]
  float* hot_sum;   // sums of those parts, then of the first parts  [2*3*hot_parts][largest slice]
};
// Items of a slice that one block adds up; the rest are parts of their own.  A block takes about 50 ns per
// item at ranks up to 32, 85 to 115 at larger ones and 400 at d1 = 20, r1 = 70: parts of 20 to 30 us each
// (700 copies of one id there: 344 us a step in parts of 512, 104 in parts of 64; the indexed kernels 103).
__host__ __device__ inline int direct_part(const Shape& s) {
  return 512 >> ((s.r1 > 32 ? 1 : 0) + (s.d1 > 8 ? 2 : 0));
}
constexpr int kDirectPartLeast = 64;
// Most parts beyond the first that the slices of a core have.  Batches of no more than two parts' items
// are not cut: listing parts and looking for them costs every batch a few per cent (700 uniform ids at
// rank 32 31.5 -> 35 us a step), and a single id 1024 times at rank 32 takes 70 us in one block, 72 on the
// indexed kernels.
inline int hot_parts(const Shape& s, int64_t items) {
  return items > 2 * direct_part(s) ? (int)(items / direct_part(s)) : 0;
}

// All device arrays carved out of the caller's workspace.
struct Workspace {
  Counters* ctr;
  uint32_t* key[2];   // radix-sort ping-pong keys      [maxB]
  uint32_t* val[2];   // radix-sort ping-pong positions [maxB]
  uint32_t* cnt;      // per-block digit histograms [sortBlocks * kMaxBins]; usually in the memory of c3_item
  uint32_t* tot;      // digit totals of the current pass  [kMaxBins]
  uint32_t* seg_nu;   // new ids per block of sorted slots      [slotBlocks]
  uint32_t* seg_nq;   // new prefixes per block of sorted slots [slotBlocks]
  int4* seg_base;     // per block of slots: its first unique id, its first prefix, how many of each
  uint16_t* seg_rows; // per block of slots: how many of these have which i3, and which i2
  int* s_u;           // sorted slot -> unique-id index (-1 for out-of-range ids) [maxB]
  int4* s_rec;        // sorted slot -> {unique-id index, batch position, prefix, i3} [maxB]
  int* u_rs;          // unique id -> first sorted slot  [maxB+1]
  int* u_i3;          // unique id -> i3                 [maxB]
  int* u_q;           // unique id -> prefix index       [maxB]
  int* u_code;        // unique id -> where its gradient row is: batch position, or -(u+1) [maxB]
  int* q_us;          // prefix -> first unique id       [maxQ+1]
  int* q_i1;          // prefix -> i1                    [maxQ]
  int* q_i2;          // prefix -> i2                    [maxQ]
  int* c3_start;      // first chunk of each i3 group [n3+1]
  int4* c3_desc;      // chunk -> {i3, 0, items, 0}  [maxChunk3]
  int4* walk3;        // columns of walk_chunks3: {first chunk of its i3, chunks, which column, of how many} [2*n3]
  int2* c3_item;      // chunk, t -> {gradient-row code, prefix} of its t-th id [maxChunk3][kChunk3]
  int* c2_start;      // [n2+1]
  int4* c2_desc;      // chunk -> {i2, 0, items, 0}  [maxChunk2]
  int4* c2_item;      // chunk, t -> {q, i1, first unique id, end} of its t-th prefix [maxChunk2][kChunk2]
  int* g1_first;      // i1 -> first prefix with that i1 (prefixes are sorted by i1) [n1]
  int* g1_end;        // i1 -> one past its last prefix; directly follows g1_first  [n1]
  float* P;           // prefix products G1[i1] G2[i2]   [maxQ][PN]
  float* gsum;        // per unique id, sum of its rows' gradients [maxB][D]
  float* carry;       // per tile: head and tail partial sums [tiles][2][D]
  float* dPsum;       // per prefix: gradient of its product  [maxQ][PN]
  float* dg1part;     // per prefix: its term of dG1[i1]      [maxQ][S1]
  float* part3;       // per chunk: partial dG3 slice         [maxChunk3][S3]
  float* part2;       // per chunk: partial dG2 slice         [maxChunk2][S2]
  DirectBuffers direct;
};

struct Plan {
  // Slab split: with d1 = 4*split (split > 1) and the other factors fit for the matrix-core
  // kernels, G1[i1] (d1 x r1) is read as split slices of 4 x r1, i.e. as a table with split*n1
  // first-core slices and d1 = 4 whose row for (split*i1 + h, i2, i3) is the h-th run of D/split
  // floats of the caller's row for (i1, i2, i3).  A batch of B ids is then a batch of split*B ids
  // of that table, out/grad [B][D] are its [split*B][D/split] arrays, and the cores are the same
  // memory.  sh, maxB and maxQ describe the table the kernels see; user_* what the caller sees.
  int split;
  bool mfma;  // the shape runs on the matrix-core kernels (and they are not switched off)
  int64_t user_maxB, user_N;
  int user_D;
  Shape sh;
  int64_t maxB, maxQ;
  int sortBlocksMax, slotBlocksMax, tilesMax;
  int64_t maxChunk3, maxChunk2;
  SortKeys keys;         // sort by table row (the batches that train)
  // Lookups at ranks up to 32 (k_lookup_mfma): caller's ids, not slabs, sorted by prefix only, and that
  // with i2 in front, so that neighbours share a G2 slice.  i3_bits = 0: other shapes.
  SortKeys lookup_keys;
  int lookup_i3_bits;
  uint32_t user_n1;
  int direct_cap;        // lookups of up to this many items take the index-free kernels (0: never)
  int direct_train_cap;  // the same for batches that backward_update follows
  // blocks of the prefix kernels for ranks 64 and 128 that the device holds at once (forward,
  // backward); asked of the runtime at the first launch, 0 until then
  mutable int unit_slots[2] = {0, 0};
};

// Chunks whose dG2 terms are added up before a partial sum is written, at the ranks of the wide
// prefix kernels: partials of 64 to 256 KiB each cost more than the products they hold, so a batch
// with many chunks takes eight per partial, one with few keeps the blocks busy instead.  A partial
// covers chunks [g*k, g*k+k) of one i2; it is written at the index of its first chunk.
constexpr int kWideGroup = 8;
__host__ __device__ inline int wide_group(int nchunk2, int r) {
  int g = 1;
  while (g < kWideGroup && nchunk2 * (r / 32) >= 4096 * g) g *= 2;
  return g;
}

enum KernelSlot {
  kSlotSortHist = 0,
  kSlotSortScan,
  kSlotSortScatter,
  kSlotSegCount,
  kSlotSegWrite,
  kSlotGroup,
  kSlotPrefixFwd,
  kSlotRowFwd,
  kSlotGsum,
  kSlotGsumFix,
  kSlotUBwd,
  kSlotDg3,
  kSlotPrefixBwd,
  kSlotSgd,
  kSlotDirectFwd,   // index-free kernels: rows, per-item gradients, sums and update
  kSlotDirectBwd,
  kSlotDirectApply,
  kSlotTable,
  kSlotLookup,
  kSlotEventPair,  // an event pair with nothing between: the cost the timing itself adds to a slot
  kSlotCount
};

__device__ __forceinline__ uint32_t key_of_id(const IdSource& src, int idx, uint32_t N) {
  int pos = idx, slab = 0;
  if (src.split > 1) {
    pos = idx / src.split;
    slab = idx - pos * src.split;
  }
  int64_t id = src.ids != nullptr ? src.ids[pos] : src.base + pos;
  if (src.reindex != nullptr) {
    // node re-indexing (paper Section 4.2: ids renumbered so that a partition's nodes are
    // consecutive): one gather in front of the split
    if ((uint64_t)id >= (uint64_t)src.n_ids) return N;
    id = src.reindex[id];
  }
  // ids outside the table (negative ones included) become the sentinel N and sort to the end
  if ((uint64_t)id >= (uint64_t)src.rows) return N;
  if (src.split > 1) {
    // first-core index i1 -> split*i1 + slab, the other two coordinates stay
    const int64_t i1 = id / src.n23;
    id += ((int64_t)(src.split - 1) * i1 + slab) * src.n23;
  }
  return (uint32_t)id;
}
__device__ __forceinline__ uint32_t key_of_id(const PrefixSource& src, int idx, uint32_t sentinel) {
  const uint32_t row = key_of_id(src.ids, idx, sentinel);
  if ((int64_t)row >= src.ids.rows) return sentinel;
  const uint32_t p = row / src.n3, i3 = row - p * src.n3, i1 = p / src.n2, i2 = p - i1 * src.n2;
  return ((i2 * src.n1 + i1) << src.i3_bits) | i3;
}

// One entry of a core under the update rule: the SGD step, the Adagrad step  S += dG^2,
// G -= lr * dG / (sqrt(S) + eps),  or the Adam step  m = b1 m + (1-b1) dG,
// v = b2 v + (1-b2) dG^2,  G -= lr * (m corr1) / (sqrt(v corr2) + eps).  St and Vt point at the
// entry's state (Adagrad sum or Adam first moment; Adam second moment).
template <int RULE>
__device__ __forceinline__ float updated_entry(float g_old, float grad, float lr, const UpdateRule& ada,
                                               float* St, float* Vt) {
  if constexpr (RULE == kUpdateAdam) {
    const float m = fmaf(ada.beta1, *St, (1.f - ada.beta1) * grad);
    const float v = fmaf(ada.beta2, *Vt, (1.f - ada.beta2) * grad * grad);
    *St = m;
    *Vt = v;
    return g_old - lr * (m * ada.corr1) / (sqrtf(v * ada.corr2) + ada.eps);
  } else if constexpr (RULE == kUpdateAdagrad) {
    const float sq = fmaf(grad, grad, *St);
    *St = sq;
    return g_old - lr * grad / (sqrtf(sq) + ada.eps);
  } else {
    return fmaf(-lr, grad, g_old);
  }
}

// Inclusive prefix sum over the wavefront: inside every row of 16 lanes with cross-lane moves in
// the vector ALU (row_shr by 1, 2, 4, 8; lanes without a source add zero), then the totals of the
// rows before a lane's own are added.
template <int BY>
__device__ __forceinline__ uint32_t row_shr_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + BY, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, int lane) {
  v += row_shr_or_zero<1>(v);
  v += row_shr_or_zero<2>(v);
  v += row_shr_or_zero<4>(v);
  v += row_shr_or_zero<8>(v);
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
  const int row = lane / 16;
  return v + (row >= 1 ? r0 : 0u) + (row >= 2 ? r1 : 0u) + (row >= 3 ? r2 : 0u);
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max(v, row_shr_or_zero<1>(v));
  v = max(v, row_shr_or_zero<2>(v));
  v = max(v, row_shr_or_zero<4>(v));
  v = max(v, row_shr_or_zero<8>(v));
  auto row = [&](int last) { return (uint32_t)__builtin_amdgcn_readlane((int)v, last); };
  return max(max(row(15), row(31)), max(row(47), row(63)));
}

// LDS writes of a wavefront become visible to its own later reads
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef float f4 __attribute__((ext_vector_type(4)));

// Transposes the 4 x 4 block that four neighbouring lanes hold a line each of.
template <int PERM>
__device__ __forceinline__ float quad_get(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), PERM, 0xf, 0xf, true));
}
__device__ __forceinline__ f4 quad_turned(f4 v, int lane) {
  const bool odd = lane & 1, upper = lane & 2;
  // 2 x 2 blocks between lanes l and l ^ 1, then the blocks between l and l ^ 2
  const float a = quad_get<0xB1>(odd ? v.x : v.y), b = quad_get<0xB1>(odd ? v.z : v.w);
  v = odd ? f4{a, v.y, b, v.w} : f4{v.x, a, v.z, b};
  const float c = quad_get<0x4E>(upper ? v.x : v.z), d = quad_get<0x4E>(upper ? v.y : v.w);
  return upper ? f4{c, d, v.z, v.w} : f4{v.x, v.y, c, d};
}

}  // namespace ttemb
