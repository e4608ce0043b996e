// Index pipeline of the TT-embedding forward pass (gfx950).
//
//   ids --split--> sort keys --stable LSD radix sort--> sorted slots
//       --segment scan--> unique ids (U) and unique (i1,i2) prefixes (Q) with their extents
//       --stable bucket passes--> unique ids grouped by i3, prefixes grouped by i2
//
// The split is i1 = i/(n2 n3), i2 = (i/n3) mod n2, i3 = i mod n3 (paper Section 4.2).  Sorting by
// the id itself makes every sharing level of the paper's Fig. "node-index" a contiguous run: equal
// ids, ids with a common (i1,i2) prefix (they share G1[i1] G2[i2]), ids with a common i1.
// Everything here is integer work and is bit-exact; all orders are stable, so the floating-point
// sums that later follow these lists are formed in a fixed order.
#include <algorithm>
#include <type_traits>

#include "tt_emb_internal.h"

namespace ttemb {

// ---------------------------------------------------------------------------------------------
// block-wide helpers; ldsw holds at least one word per wavefront of the block

// Exclusive prefix of v over the block's threads; *total receives the block sum.
__device__ __forceinline__ uint32_t block_exclusive_scan_value(uint32_t v, uint32_t* ldsw,
                                                               uint32_t* total) {
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave, nw = blockDim.x / kWave;
  const uint32_t incl = wave_inclusive_scan(v, lane);
  if (lane == kWave - 1) ldsw[w] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int k = 0; k < nw; ++k) {
    const uint32_t t = ldsw[k];
    base += (k < w) ? t : 0u;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return base + incl - v;
}

// In-place exclusive scan of an LDS array arr[0..n), n <= kMaxBins; returns the total.
__device__ uint32_t block_exclusive_scan(uint32_t* arr, int n, uint32_t* ldsw) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int per = (n + nt - 1) / nt;
  const int lo = min(tid * per, n), hi = min(lo + per, n);
  uint32_t s = 0;
  for (int i = lo; i < hi; ++i) s += arr[i];
  uint32_t total;
  uint32_t run = block_exclusive_scan_value(s, ldsw, &total);
  for (int i = lo; i < hi; ++i) {
    const uint32_t t = arr[i];
    arr[i] = run;
    run += t;
  }
  __syncthreads();
  return total;
}

// Lanes of a wavefront that hold the same digit (among lanes with valid set).  One ballot per bit of
// the widest digit (higher bits are zero everywhere and cost nothing but their ballot): a lane
// collects the lanes that differ from it in some bit as (vote xor own bit replicated).
constexpr int kMaxBits = 11;
static_assert((1 << kMaxBits) == kMaxBins, "digits have at most kMaxBits bits");
__device__ __forceinline__ unsigned long long match_digit(int digit, bool valid) {
  const int d = valid ? digit : 0;
  uint32_t lo = 0u, hi = 0u;
#pragma unroll
  for (int bit = 0; bit < kMaxBits; ++bit) {
    const int t = (d << (31 - bit)) >> 31;  // 0 or -1
    const unsigned long long vote = __ballot(t < 0);
    lo |= (uint32_t)vote ^ (uint32_t)t;
    hi |= (uint32_t)(vote >> 32) ^ (uint32_t)t;
  }
  return ~(((unsigned long long)hi << 32) | lo) & __ballot(valid);
}

constexpr int kSteps = kSortWaveItems / kWave;  // most items per lane
static_assert((kChunk2 & (kChunk2 - 1)) == 0 && (kChunk3 & (kChunk3 - 1)) == 0 &&
                  (kChunk3Min & (kChunk3Min - 1)) == 0,
              "chunk sizes are powers of two: positions inside a bucket are cut with shifts");

// Column sums over the rows of 16-bit bucket counts that the nblk blocks of a pass left, `stride` counts
// apart: per bucket the items of all blocks (tot) and those of blocks before blk (before).  Eight buckets are
// one 16-byte load (`words` of them a row), so a row takes few threads, and the threads are dealt over the
// rows too, ROWS of them a thread under way at once, where one thread per bucket makes a chain of the rows.  No more
// threads than that takes: their sums meet in LDS, and every further one is another atomic on the same words
// (200,000 ids, 1024 threads in the grouping kernel: 176 us a step with all of them, 172 without).
template <int ROWS>  // rows a thread has in flight
struct ColumnSums {
  uint32_t t8[8], b8[8];
  int at;  // this thread's word of a row, or -1
  __device__ __forceinline__ void load(const uint16_t* __restrict__ rows, int stride, int words, int nblk, int blk) {
    const int groups = min((int)blockDim.x / words, (nblk + ROWS - 1) / ROWS), g = (int)threadIdx.x / words;
    at = g < groups ? (int)threadIdx.x - g * words : -1;
#pragma unroll
    for (int j = 0; j < 8; ++j) t8[j] = b8[j] = 0u;
    if (at < 0) return;
    const uint4* col = (const uint4*)rows + at;
    const int stride4 = stride / 8;
    for (int r0 = g; r0 < nblk; r0 += groups * ROWS) {
      uint4 v[ROWS];
#pragma unroll
      for (int k = 0; k < ROWS; ++k) v[k] = col[(size_t)min(r0 + k * groups, nblk - 1) * stride4];
      __builtin_amdgcn_sched_barrier(0);
      // Eight rows are added two counts to a word: eight times at most 4096 items stay below 2^16.
#pragma unroll
      for (int k0 = 0; k0 < ROWS; k0 += 8) {
        uint32_t t[4] = {}, b[4] = {};
#pragma unroll
        for (int k = k0; k < k0 + 8; ++k) {
          const int r = r0 + k * groups;
          const uint32_t x[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            t[j] += r < nblk ? x[j] : 0u;
            b[j] += r < blk ? x[j] : 0u;
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          t8[2 * j] += t[j] & 0xffffu;
          t8[2 * j + 1] += t[j] >> 16;
          b8[2 * j] += b[j] & 0xffffu;
          b8[2 * j + 1] += b[j] >> 16;
        }
      }
    }
  }
  // tot and before have been cleared, with a barrier behind it; the caller's next barrier ends the sums
  __device__ __forceinline__ void add_to(uint32_t* tot, uint32_t* before) const {
    if (at < 0) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (t8[j] != 0) atomicAdd(&tot[at * 8 + j], t8[j]);
      if (b8[j] != 0) atomicAdd(&before[at * 8 + j], b8[j]);
    }
  }
};

// Stable ranks of a block's items in their buckets, given to take(step, rank).  Every wavefront holds up to 256 consecutive items,
// 64 a step (digit -1: no item); the wavefronts' runs follow each other.  wh: a row per wavefront, stride words
// apart, of row_words words (both multiples of four), two 16-bit buckets a word: a wavefront owns 256 items and a
// block at most 4096, so both fit.
template <int NT, class F>
__device__ __forceinline__ void block_ranks(uint32_t* wh, int stride, int row_words, const int (&digits)[kSteps],
                                            F take) {
  const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
  uint32_t* mine = wh + w * stride;
  // every wavefront clears its own counters, 16 bytes per lane and write (no barrier: nobody else
  // touches them before the next one)
  for (int i = lane; i < row_words / 4; i += kWave) ((uint4*)mine)[i] = make_uint4(0u, 0u, 0u, 0u);

  // Each wavefront walks its items in order, 64 at a time.  Lanes holding the same digit find each
  // other by ballots; the lowest of them advances the wavefront's bucket counter for all, which
  // gives every item its rank among the wavefront's items of that bucket.
  uint32_t rank[kSteps];
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  unsigned long long peers[kSteps];
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const bool valid = digits[step] >= 0;
    peers[step] = 0ull;
    if (__ballot(valid) != 0ull) peers[step] = match_digit(digits[step], valid);  // wave-uniform
  }
  // the counter updates of the steps go out back to back (the LDS keeps a wavefront's atomics in
  // program order, which is what makes the ranks stable), their results are picked up afterwards
  uint32_t old[kSteps];
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const int digit = digits[step];
    old[step] = 0;
    if (digit >= 0 && lane == __ffsll((long long)peers[step]) - 1)
      old[step] = atomicAdd(&mine[digit >> 1], (uint32_t)__popcll(peers[step]) << (16 * (digit & 1)));
  }
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const int digit = digits[step];
    const int leader = digit >= 0 ? (__ffsll((long long)peers[step]) - 1) : lane;
    rank[step] = ((__shfl(old[step], leader) >> (16 * (digit & 1))) & 0xffffu) +
                 (uint32_t)__popcll(peers[step] & lt_mask);
  }
  __syncthreads();
  // per bucket: counts of the wavefronts -> offsets inside the block (one thread per word)
  for (int word = tid; word < row_words; word += NT) {
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int k = 0; k < NT / kWave; ++k) {
      const uint32_t c = wh[k * stride + word];
      wh[k * stride + word] = lo | (hi << 16);
      lo += c & 0xffffu;
      hi += c >> 16;
    }
  }
  __syncthreads();
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const int digit = digits[step];
    if (digit >= 0) take(step, rank[step] + ((mine[digit >> 1] >> (16 * (digit & 1))) & 0xffffu));
  }
}

template <int NT, bool FOLDS>
struct alignas(16) ScatterLds {
  uint32_t wh[NT / kWave][kMaxBins / 2];  // counters of block_ranks
  uint32_t tot[kMaxBins];                 // bucket totals, then this block's first output per bucket
  uint32_t before[FOLDS ? kMaxBins : 1];  // items of earlier blocks per bucket
  uint32_t ldsw[NT / kWave];
};

// One block's share of a stable counting-sort pass over n_items items (block blk of NT threads owns
// items [blk*4*NT, +4*NT), each of its wavefronts 256 of them in order).  FOLDS: cnt holds the blocks'
// own histograms as rows of 16-bit counts, and every block adds up its columns itself; else cnt[b][bin]
// holds, per bucket, the items of blocks before b and tot[bin] the bucket totals (both from a
// column-scan kernel over the blocks' histograms).
// ItemOps: Item load(int idx); int digit(Item); void emit(uint32_t pos, Item).
template <int NT, bool FOLDS, class ItemOps>
__device__ void stable_scatter_block(ScatterLds<NT, FOLDS>& L, int blk, int nblk, int n_items, int bins,
                                     const uint32_t* __restrict__ cnt,
                                     const uint32_t* __restrict__ tot, ItemOps ops) {
  constexpr int kItems = sort_items(NT);
  const int tid = threadIdx.x;

  // items first: their loads overlap the table work below
  const int w = tid / kWave, lane = tid % kWave;
  const int wbase = blk * kItems + w * kSortWaveItems;
  typename ItemOps::Item items[kSteps];
  int digits[kSteps];
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const int idx = wbase + step * kWave + lane;
    items[step] = ops.load(idx < n_items ? idx : 0);
  }
  uint32_t earlier[kMaxBins / NT];  // items of my buckets in earlier blocks
  if constexpr (!FOLDS) {
    uint32_t total[kMaxBins / NT];
#pragma unroll
    for (int k = 0; k < kMaxBins / NT; ++k) {
      const int bc = min(tid + k * NT, bins - 1);
      total[k] = tot[bc];
      earlier[k] = cnt[(size_t)blk * bins + bc];
    }
#pragma unroll
    for (int k = 0; k < kMaxBins / NT; ++k)
      if (tid + k * NT < bins) L.tot[tid + k * NT] = total[k];
  } else {
    const int words = sort_row_words(bins);
    ColumnSums<NT == 256 ? 32 : 16> sums;
    sums.load((const uint16_t*)cnt, words * 8, words, nblk, blk);
    for (int i = tid; i < words * 8; i += NT) L.tot[i] = L.before[i] = 0u;
    __syncthreads();
    sums.add_to(L.tot, L.before);
  }
  __builtin_amdgcn_sched_barrier(0);  // keep the loads together: their latencies overlap
#pragma unroll
  for (int step = 0; step < kSteps; ++step) digits[step] = ops.digit(items[step]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int step = 0; step < kSteps; ++step)
    if (wbase + step * kWave + lane >= n_items) digits[step] = -1;
  __syncthreads();
  block_exclusive_scan(L.tot, bins, L.ldsw);
#pragma unroll
  for (int k = 0; k < kMaxBins / NT; ++k) {
    const int bin = tid + k * NT;
    if (bin < bins) {
      if constexpr (FOLDS) L.tot[bin] += L.before[bin];
      else L.tot[bin] += earlier[k];
    }
  }
  block_ranks<NT>(&L.wh[0][0], kMaxBins / 2, max((bins / 2 + 3) & ~3, 4), digits,
                  [&](int step, uint32_t rank) { ops.emit(L.tot[digits[step]] + rank, items[step]); });
}

// ---------------------------------------------------------------------------------------------
// LSD radix sort of (key = id or sentinel, value = batch position)

struct KV {
  uint32_t key, val;
};

template <bool FIRST>
struct SortOps {
  using Item = KV;
  const uint32_t* kin;
  const uint32_t* vin;
  uint32_t* kout;
  uint32_t* vout;
  int shift;
  uint32_t mask;
  __device__ Item load(int idx) const { return KV{kin[idx], FIRST ? (uint32_t)idx : vin[idx]}; }
  __device__ int digit(Item it) const { return (int)((it.key >> shift) & mask); }
  __device__ void emit(uint32_t pos, Item it) const {
    kout[pos] = it.key;
    vout[pos] = it.val;
  }
};

struct KeysInPlace {};  // source of the passes behind the first

// Bucket counts of one radix digit per block of sort_items(NT) items.  Equal digits inside a
// wavefront step are counted with one LDS atomic (a hot id would otherwise serialise thousands of
// them).  The first pass also clears the tables that later kernels of the same forward add into, and
// leaves the keys for its scatter, which need not split and renumber the ids again.
template <int NT, class SRC>
__global__ __launch_bounds__(NT) void k_sort_hist(
    SRC src, uint32_t* keys_io, int B, uint32_t N, int shift,
    int bits, bool folds, uint32_t* __restrict__ cnt, uint32_t* zero, int zero_n, Counters* ctr) {
  constexpr bool FROM_IDS = !std::is_same_v<SRC, KeysInPlace>;
  __shared__ uint32_t h[kMaxBins];
  const int tid = threadIdx.x, bins = 1 << bits;
  const uint32_t mask = (uint32_t)bins - 1u;
  const int w = tid / kWave, lane = tid % kWave;
  const int wbase = blockIdx.x * sort_items(NT) + w * kSortWaveItems;
  uint32_t keys[kSteps];
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const int idx = wbase + step * kWave + lane;
    const int ic = min(idx, B - 1);
    if constexpr (FROM_IDS) keys[step] = key_of_id(src, ic, N);
    else keys[step] = keys_io[ic];
  }
  __builtin_amdgcn_sched_barrier(0);  // keep the loads together: their latencies overlap
  if (FROM_IDS) {
#pragma unroll
    for (int step = 0; step < kSteps; ++step) {
      const int idx = wbase + step * kWave + lane;
      if (idx < B) keys_io[idx] = keys[step];
    }
    const int gtid = blockIdx.x * NT + tid, gn = gridDim.x * NT;
    for (int i = gtid; i < zero_n; i += gn) zero[i] = 0u;
    if (gtid == 0) {
      ctr->err = 0;
      ctr->n_split = 0;
      ctr->small = 0;
    }
  }
  const int padded = sort_row_words(bins) * 8;
  for (int i = tid; i < padded; i += NT) h[i] = 0u;
  __syncthreads();
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const int idx = wbase + step * kWave + lane;
    const bool valid = idx < B;
    if (__ballot(valid) == 0ull) continue;
    const int digit = (int)((keys[step] >> shift) & mask);
    const unsigned long long peers = match_digit(digit, valid);
    if (valid && lane == __ffsll((long long)peers) - 1)
      atomicAdd(&h[digit], (uint32_t)__popcll(peers));
  }
  __syncthreads();
  if (folds) {  // a row of 16-bit counts (a block has at most 4096 items)
    uint32_t* row = cnt + (size_t)blockIdx.x * (padded / 2);
    for (int i = tid; i < padded / 2; i += NT) row[i] = h[2 * i] | (h[2 * i + 1] << 16);
  } else {
    for (int i = tid; i < bins; i += NT) cnt[(size_t)blockIdx.x * bins + i] = h[i];
  }
}

template <int NT, bool FROM_IDS, bool FOLDS>
__global__ __launch_bounds__(NT) void k_sort_scatter(SortOps<FROM_IDS> ops, int B,
                                                               int bits,
                                                               const uint32_t* __restrict__ cnt,
                                                               const uint32_t* __restrict__ tot) {
  __shared__ ScatterLds<NT, FOLDS> L;
  stable_scatter_block<NT, FOLDS>(L, (int)blockIdx.x, (int)gridDim.x, B, 1 << bits, cnt, tot, ops);
}

// Turns the blocks' bucket counts cnt[b][bin] into counts of earlier blocks (exclusive scan down
// each column) and leaves the column totals in tot[bin].  A block takes 32 buckets (128 bytes of a
// row) and cuts the rows into 32 runs, one thread per bucket and run: a column of up to 256 rows is
// eight loads in flight per thread, where one thread per column made a chain of them.
constexpr int kScanThreads = 1024, kScanBins = 32, kScanRuns = kScanThreads / kScanBins;
constexpr int kScanRows = 8;  // rows of a run that stay in registers
__global__ __launch_bounds__(kScanThreads) void k_sort_colscan(uint32_t* __restrict__ cnt,
                                                               uint32_t* __restrict__ tot, int nblk,
                                                               int bins) {
  __shared__ uint32_t part[kScanRuns][kScanBins];
  const int b = threadIdx.x % kScanBins, run = threadIdx.x / kScanBins;
  const int bin = blockIdx.x * kScanBins + b;
  const int per = (nblk + kScanRuns - 1) / kScanRuns;
  const int lo = min(run * per, nblk), hi = min(lo + per, nblk);
  uint32_t* col = cnt + min(bin, bins - 1);
  uint32_t c[kScanRows];
  uint32_t sum = 0;
  for (int r0 = lo; r0 < hi; r0 += kScanRows) {
#pragma unroll
    for (int k = 0; k < kScanRows; ++k) c[k] = col[(size_t)min(r0 + k, hi - 1) * bins];
#pragma unroll
    for (int k = 0; k < kScanRows; ++k) sum += r0 + k < hi ? c[k] : 0u;
  }
  part[run][b] = sum;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int k = 0; k < kScanRuns; ++k) {
    const uint32_t v = part[k][b];
    before += k < run ? v : 0u;
    total += v;
  }
  if (bin >= bins) return;
  if (run == 0) tot[bin] = total;
  for (int r0 = lo; r0 < hi; r0 += kScanRows) {
    if (per > kScanRows) {  // a longer run is read again
#pragma unroll
      for (int k = 0; k < kScanRows; ++k) c[k] = col[(size_t)min(r0 + k, hi - 1) * bins];
    }
#pragma unroll
    for (int k = 0; k < kScanRows; ++k) {
      if (r0 + k < hi) col[(size_t)(r0 + k) * bins] = before;
      before += c[k];
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Segment discovery over the sorted keys

// What a sorted slot begins and ends.
struct SlotFlags {
  uint32_t key, prev;
  bool valid, newu, newq, last_valid, single, split;
};

__device__ __forceinline__ SlotFlags slot_flags(const uint32_t* __restrict__ skey, int B, uint32_t N,
                                                uint32_t n3, int s) {
  SlotFlags f;
  const uint32_t key = s < B ? skey[s] : 0xffffffffu;
  const uint32_t prev = s > 0 && s - 1 < B ? skey[s - 1] : 0xffffffffu;
  const uint32_t next = s + 1 < B ? skey[s + 1] : 0xffffffffu;
  f.key = key;
  f.prev = prev;
  f.valid = (s < B) && (key < N);
  const bool first = (s == 0);
  // a new entry: a new id, or the next kEntrySlots piece of a long run of one id
  const bool cut = (s % kEntrySlots) == 0;
  f.newu = f.valid && (first || key != prev || cut);
  f.split = f.valid && !first && key == prev && cut;
  f.newq = f.valid && (first || (key / n3) != (prev / n3));
  f.last_valid = f.valid && !(next < N);
  // the entry holds exactly one slot: its gradient row is read where it lies
  f.single = f.newu && (next != key || ((s + 1) % kEntrySlots) == 0);
  return f;
}

constexpr int kSegThreads = 1024;
// A wavefront of the segment kernels owns ITEMS * 64 consecutive slots, 64 a step, so that what a step
// loads and stores lies together.
template <int ITEMS>
__device__ __forceinline__ int first_slot() {
  return ((int)(blockIdx.x * kSegThreads + threadIdx.x) / kWave * ITEMS) * kWave + (int)threadIdx.x % kWave;
}

// New ids and prefixes of every block of 1024*ITEMS sorted slots.
template <int ITEMS>
__global__ __launch_bounds__(kSegThreads) void k_seg_count(const uint32_t* __restrict__ skey, int B, uint32_t N,
                                                  uint32_t n3, uint32_t* __restrict__ seg_nu,
                                                  uint32_t* __restrict__ seg_nq) {
  __shared__ uint32_t ldsw[kSegThreads / kWave];
  const int s0 = first_slot<ITEMS>();
  uint32_t c = 0;  // new ids in the upper half, new prefixes in the lower
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const SlotFlags f = slot_flags(skey, B, N, n3, s0 + j * kWave);
    c += ((uint32_t)__popcll(__ballot(f.newu)) << 16) + (uint32_t)__popcll(__ballot(f.newq));
  }
  if (threadIdx.x % kWave == 0) ldsw[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
#pragma unroll
    for (int k = 0; k < kSegThreads / kWave; ++k) total += ldsw[k];
    seg_nu[blockIdx.x] = total >> 16;
    seg_nq[blockIdx.x] = total & 0xffffu;
  }
}

// Numbers the unique ids and prefixes in sorted order, records their extents and coordinates, and leaves
// for the grouping pass, per block of 1024*ITEMS slots, which ids and prefixes are its own (seg_base: first
// id, first prefix, how many of each) and how many of them have which i3 resp. i2 (a row of p3 + p2 16-bit
// counts).  The counts are made in LDS: added to tables in memory, one atomic per new id and prefix, they
// were most of this kernel (two a slot at worst; a compute unit retires one lane's atomic in 16 cycles):
// 100,000 uniform items of n3 = 56 8.3 -> 5.1 us, a million Zipf items of n3 = 500 33 -> 16.
// u_code[u] says where the gradient row of unique id u will be found: >= 0 is the batch position
// of its only occurrence, -(u+1) means "row u of the per-id sums".
template <int ITEMS>
__global__ __launch_bounds__(kSegThreads) void k_seg_write(
    const uint32_t* __restrict__ skey, const uint32_t* __restrict__ perm, int B, Shape sh, int p3, int p2,
    const uint32_t* __restrict__ seg_nu, const uint32_t* __restrict__ seg_nq, int* __restrict__ s_u,
    int4* __restrict__ s_rec, int* __restrict__ u_rs, int* __restrict__ u_i3, int* __restrict__ u_q, int* __restrict__ u_code,
    int* __restrict__ q_us, int* __restrict__ q_i1, int* __restrict__ q_i2, int4* __restrict__ seg_base,
    uint16_t* __restrict__ rows, int* __restrict__ g1_first, int* __restrict__ g1_end,
    Counters* __restrict__ ctr) {
  extern __shared__ uint32_t seg_hist[];  // p3 + p2 counters
  __shared__ uint32_t ldsw[3][kSegThreads / kWave];
  const int tid = threadIdx.x, blk = blockIdx.x, lane = tid % kWave, w = tid / kWave;
  const int s0 = first_slot<ITEMS>();
  SlotFlags f[ITEMS];
  uint32_t bpos[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    f[j] = slot_flags(skey, B, sh.N, sh.n3, s0 + j * kWave);
    bpos[j] = perm[min(s0 + j * kWave, B - 1)];
  }
  uint32_t pu = 0, pq = 0;  // ids and prefixes of the blocks before
  for (int b2 = tid; b2 < blk; b2 += kSegThreads) {
    pu += seg_nu[b2];
    pq += seg_nq[b2];
  }
  for (int i = tid; i < p3 + p2; i += kSegThreads) seg_hist[i] = 0u;
  uint32_t c = 0;  // new ids in the upper half, new prefixes in the lower
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    c += ((uint32_t)__popcll(__ballot(f[j].newu)) << 16) + (uint32_t)__popcll(__ballot(f[j].newq));
  pu = wave_inclusive_scan(pu, lane);
  pq = wave_inclusive_scan(pq, lane);
  if (lane == kWave - 1) {
    ldsw[0][w] = c;
    ldsw[1][w] = pu;
    ldsw[2][w] = pq;
  }
  __syncthreads();
  uint32_t mine = 0, here = 0, ru = 0, rq = 0;
#pragma unroll
  for (int k = 0; k < kSegThreads / kWave; ++k) {
    const uint32_t v = ldsw[0][k];
    mine += k < w ? v : 0u;
    here += v;
    ru += ldsw[1][k];
    rq += ldsw[2][k];
  }
  if (tid == 0) seg_base[blk] = make_int4((int)ru, (int)rq, (int)(here >> 16), (int)(here & 0xffffu));
  ru += mine >> 16;  // unique ids before the wavefront's slots
  rq += mine & 0xffffu;

  if (blk == 0 && tid == 0 && !f[0].valid) {  // no in-range id at all
    ctr->U = 0;
    ctr->Q = 0;
    ctr->nvalid = 0;
    u_rs[0] = 0;
    q_us[0] = 0;
  }
  const unsigned long long up_to = ~0ull >> (kWave - 1 - lane);  // this lane and those below
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int s = s0 + j * kWave;
    const unsigned long long mu = __ballot(f[j].newu), mq = __ballot(f[j].newq);
    const int u = (int)(ru + __popcll(mu & up_to)) - 1, q = (int)(rq + __popcll(mq & up_to)) - 1;
    ru += __popcll(mu);
    rq += __popcll(mq);
    if (s >= B) continue;
    if (!f[j].valid) {
      s_u[s] = -1;
      s_rec[s] = make_int4(-1, (int)bpos[j], 0, 0);
      continue;
    }
    s_u[s] = u;
    const uint32_t k = f[j].key, p = k / sh.n3, i3 = k - p * sh.n3;  // p: prefix number i1*n2 + i2
    // everything the row kernel needs about a slot in one record (one load instead of a chain)
    s_rec[s] = make_int4(u, (int)bpos[j], q, (int)i3);
    if (f[j].split) atomicAdd(&ctr->n_split, 1);
    if (f[j].newu) {
      u_rs[u] = s;
      u_i3[u] = (int)i3;
      u_q[u] = q;
      u_code[u] = f[j].single ? (int)bpos[j] : -(u + 1);
      atomicAdd(&seg_hist[i3], 1u);
    }
    if (f[j].newq) {
      const uint32_t i1 = p / sh.n2, i2 = p - i1 * sh.n2;
      q_us[q] = u;
      q_i1[q] = (int)i1;
      q_i2[q] = (int)i2;
      atomicAdd(&seg_hist[p3 + i2], 1u);
      // prefixes are numbered in (i1,i2) order: an i1 owns prefixes [g1_first, g1_end)
      const uint32_t i1_before = (s == 0) ? 0xffffffffu : f[j].prev / sh.n3 / sh.n2;
      if (i1_before != i1) {
        g1_first[i1] = q;
        if (s != 0) g1_end[i1_before] = q;
      }
    }
    if (f[j].last_valid) {
      ctr->U = u + 1;
      ctr->Q = q + 1;
      ctr->nvalid = s + 1;
      u_rs[u + 1] = s + 1;
      q_us[q + 1] = u + 1;
      g1_end[p / sh.n2] = q + 1;
    }
  }
  __syncthreads();
  uint32_t* row = (uint32_t*)(rows + (size_t)blk * (p3 + p2));
  for (int i = tid; i < (p3 + p2) / 2; i += kSegThreads) row[i] = seg_hist[2 * i] | (seg_hist[2 * i + 1] << 16);
}

// ---------------------------------------------------------------------------------------------
// Grouping: unique ids by i3 (for the G3 gradient), prefixes by i2 (for G2 and the prefix product).
// Only the chunks are written: per chunk a descriptor and a table of the items' records, so that the
// gradient kernels need no further look-ups.

// Unique ids by i3; chunk records are {gradient-row code, prefix}.
struct GroupOps3 {
  struct Item {
    int i3, code, q;
  };
  const int* u_i3;
  const int* u_code;
  const int* u_q;
  int2* item;
  __device__ Item load(int idx) const { return Item{u_i3[idx], u_code[idx], u_q[idx]}; }
  __device__ int digit(Item it) const { return it.i3; }
  __device__ void emit(uint32_t chunk, uint32_t t, Item it) const {
    item[(size_t)chunk * kChunk3 + t] = make_int2(it.code, it.q);
  }
};

// Prefixes by i2; chunk records are {prefix, i1, first unique id, one past its last unique id}.
struct GroupOps2 {
  struct Item {
    int q, i2, i1, u0, u1;
  };
  const int* q_i2;
  const int* q_i1;
  const int* q_us;
  int4* item;
  __device__ Item load(int idx) const {
    return Item{idx, q_i2[idx], q_i1[idx], q_us[idx], q_us[idx + 1]};
  }
  __device__ int digit(Item it) const { return it.i2; }
  __device__ void emit(uint32_t chunk, uint32_t t, Item it) const {
    item[(size_t)chunk * kChunk2 + t] = make_int4(it.q, it.i1, it.u0, it.u1);
  }
};

// LDS of a grouping block: counters of block_ranks, then three tables of one word per bucket.
__host__ __device__ constexpr int group_row_words(int bins) { return (bins + 7) / 8 * 4; }
constexpr size_t group_lds(int threads, int bins) {
  return (size_t)(threads / kWave) * group_row_words(bins) * 4 + 3 * (size_t)((bins + 7) / 8 * 8) * 4;
}

// One block's share of a stable counting-sort pass: items [first, first + count), those that slot block
// blk of nblk found.  rows: 16-bit counts per bucket of every block, `stride` apart.  Every bucket is cut
// into chunks of `chunk` items (a power of two): chunk_desc[c] = {bucket, 0, item count, 0} for all chunks
// c in bucket order, chunk_starts[bucket] the first chunk of each bucket (bins+1 entries), *n_chunks the
// number of chunks; the item that is the t-th of chunk c goes to emit(c, t, item).  Block `publisher` writes the
// tables of one entry per bucket; with walk (2*bins entries) also the columns of walk_chunks3.
// The blocks add up the columns of `rows` themselves (ColumnSums): k_group, 100,000 uniform items of n3 = 56
// 17 -> 7.4 us, 200,000 Zipf ids of n3 = 136 14.8 -> 8, 500,000 of n3 = 480 25.7 -> 15.5.
template <int NT, class ItemOps>
__device__ void group_block(int blk, int nblk, int first, int count, int bins,
                            const uint16_t* __restrict__ rows, int stride, ItemOps ops, int chunk,
                            int publisher, int* chunk_starts, int4* chunk_desc, int* n_chunks, int4* walk,
                            int* walk_cols, int* walk_steps) {
  extern __shared__ __attribute__((aligned(16))) uint32_t group_words[];
  __shared__ uint32_t ldsw[NT / kWave], most_chunks, filled;
  const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
  const int words = (bins + 7) / 8, row_words = group_row_words(bins);
  uint32_t* wh = group_words;
  uint32_t* tot = wh + (NT / kWave) * row_words;  // items per bucket
  uint32_t* before = tot + words * 8;             // those of earlier blocks
  uint32_t* aux = before + words * 8;             // chunks per bucket, then first chunk per bucket
  const int chunk_sh = 31 - __clz(chunk);
  // items first: their loads overlap the table work below
  const int per = (count + NT - 1) / NT;  // steps, so that all wavefronts have a share
  const int wbase = w * per * kWave;
  typename ItemOps::Item items[kSteps];
  int digits[kSteps];
#pragma unroll
  for (int step = 0; step < kSteps; ++step) {
    const int i = wbase + step * kWave + lane;
    items[step] = ops.load(max(first + min(i, count - 1), 0));
  }
  ColumnSums<8> sums;
  sums.load(rows, stride, words, nblk, count > 0 ? blk : 0);  // without items, nothing of the blocks before
  for (int i = tid; i < words * 16; i += NT) tot[i] = 0u;  // tot and before
#pragma unroll
  for (int step = 0; step < kSteps; ++step) digits[step] = ops.digit(items[step]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int step = 0; step < kSteps; ++step)
    if (step >= per || wbase + step * kWave + lane >= count) digits[step] = -1;
  __syncthreads();
  sums.add_to(tot, before);
  if (tid == 0) most_chunks = filled = 0u;
  __syncthreads();
  uint32_t my_most = 0, my_filled = 0;
  for (int bin = tid; bin < bins; bin += NT) {
    aux[bin] = (tot[bin] + chunk - 1) >> chunk_sh;
    my_most = max(my_most, aux[bin]);
    my_filled += aux[bin] > 0;
  }
  if (blk == publisher && walk != nullptr) {
    my_most = wave_max(my_most);
    my_filled = wave_inclusive_scan(my_filled, lane);
    if (lane == kWave - 1) {
      atomicMax(&most_chunks, my_most);
      atomicAdd(&filled, my_filled);
    }
  }
  __syncthreads();
  const uint32_t total_chunks = block_exclusive_scan(aux, bins, ldsw);
  if (blk == publisher) {
    for (int bin = tid; bin < bins; bin += NT) chunk_starts[bin] = (int)aux[bin];
    if (tid == 0) {
      chunk_starts[bins] = (int)total_chunks;
      *n_chunks = (int)total_chunks;
    }
    if (walk != nullptr) {
      auto chunks_of = [&](int bin) { return (int)((bin + 1 < bins ? aux[bin + 1] : total_chunks) - aux[bin]); };
      const uint32_t longest = (most_chunks + kXcds - 1) / kXcds;  // of the buckets' eighths
      uint32_t cols = 0, steps = longest;
      if (total_chunks >= (uint32_t)(kWalkLeast * kXcds) * filled) {
        if (bins < 2 * (int)filled && longest * bins <= kWalkMeans * (total_chunks / kXcds + bins)) {
          // a column each, also for the empty ones
          cols = (uint32_t)bins;
          for (int bin = tid; bin < bins; bin += NT) walk[bin] = make_int4((int)aux[bin], chunks_of(bin), 0, 1);
        } else {
          steps = max(kWalkMeans * ((total_chunks + kXcds * bins - 1) / (kXcds * bins)), 1u);
          uint32_t* first_col = wh;  // free until block_ranks; at least two words a bucket
          for (int bin = tid; bin < bins; bin += NT)
            first_col[bin] = ((chunks_of(bin) + kXcds - 1) / kXcds + steps - 1) / steps;
          __syncthreads();
          cols = block_exclusive_scan(first_col, bins, ldsw);
          for (int bin = tid; bin < bins; bin += NT) {
            const int first = (int)first_col[bin], n = (int)(bin + 1 < bins ? first_col[bin + 1] : cols) - first;
            for (int k = 0; k < n; ++k) walk[first + k] = make_int4((int)aux[bin], chunks_of(bin), k, n);
          }
          __syncthreads();  // block_ranks clears what the columns were counted in
        }
      }
      if (tid == 0) {
        *walk_cols = (int)cols;
        *walk_steps = (int)steps;
      }
    }
  }
  // every block of slots takes a share of the chunk descriptors
  for (uint32_t c = (uint32_t)blk * NT + tid; blk < nblk && c < total_chunks; c += (uint32_t)nblk * NT) {
    int lo = 0, hi = bins;  // last bucket whose first chunk is <= c
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (aux[mid] <= c) lo = mid; else hi = mid;
    }
    chunk_desc[c] = make_int4(lo, 0, (int)min((uint32_t)chunk, tot[lo] - (c - aux[lo]) * (uint32_t)chunk), 0);
  }
  if (count == 0) return;  // uniform for the whole block
  block_ranks<NT>(wh, row_words, row_words, digits, [&](int step, uint32_t rank) {
    const uint32_t in_bucket = before[digits[step]] + rank;
    ops.emit(aux[digits[step]] + (in_bucket >> chunk_sh), in_bucket & (uint32_t)(chunk - 1), items[step]);
  });
}

// Blocks [0, ub): unique ids by i3, first one that only writes the tables of one entry per bucket, then a block per
// block of slots; the nblk behind those: prefixes by i2.
template <int NT>
__global__ __launch_bounds__(NT) void k_group(
    Shape sh, int ub, int nblk, int chunk3, int p3, int p2, const int4* __restrict__ seg_base,
    const uint16_t* __restrict__ rows, const int* __restrict__ u_i3, const int* __restrict__ u_code,
    const int* __restrict__ u_q, const int* __restrict__ q_i2, const int* __restrict__ q_i1,
    const int* __restrict__ q_us, int* c3_start, int4* c3_desc, int2* c3_item, int* c2_start, int4* c2_desc,
    int4* c2_item, int4* walk3, Counters* ctr) {
  const bool ids = (int)blockIdx.x < ub;
  const int blk = !ids ? blockIdx.x - ub : blockIdx.x == 0 ? nblk : blockIdx.x - 1;
  const int4 base = blk < nblk ? seg_base[blk] : make_int4(0, 0, 0, 0);
  if (ids) {
    GroupOps3 ops{u_i3, u_code, u_q, c3_item};
    group_block<NT>(blk, nblk, base.x, base.z, (int)sh.n3, rows, p3 + p2, ops, chunk3, nblk, c3_start, c3_desc,
                    &ctr->nchunk3, walk3, &ctr->walk_cols, &ctr->walk_steps);
  } else {
    GroupOps2 ops{q_i2, q_i1, q_us, c2_item};
    group_block<NT>(blk, nblk, base.y, base.w, (int)sh.n2, rows + p3, p3 + p2, ops, kChunk2, 0, c2_start,
                    c2_desc, &ctr->nchunk2, nullptr, nullptr, nullptr);
  }
}

// ---------------------------------------------------------------------------------------------
// host-side launchers

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// One of the three kernels of a pass.  clear: the first one also clears the tables that the steps
// behind the sort add into (lookups have none).
template <int NT>
static void sort_pass(const Plan& pl, const Workspace& ws, const SortKeys& sk, const IdSource& src, int B,
                      int pass, bool beside, bool clear, hipStream_t st, int which) {
  const int blocks = cdiv(B, sort_items(NT));
  const int shift = sk.low + pass * sk.per;
  const int bits = sk.bits_of(pass);
  const bool folds = sort_folds(sk, B, pass, beside);
  const int in = (pass + 1) & 1;
  uint32_t *kin = ws.key[in], *vin = ws.val[in], *kout = ws.key[in ^ 1], *vout = ws.val[in ^ 1];
  if (which == 2) {
    k_sort_colscan<<<cdiv(1 << bits, kScanBins), kScanThreads, 0, st>>>(ws.cnt, ws.tot, blocks,
                                                                       1 << bits);
  } else if (which == 0) {
    auto first = [&](auto from) {
      k_sort_hist<NT><<<blocks, NT, 0, st>>>(
          from, kin, B, sk.sentinel, shift, bits, folds, ws.cnt, (uint32_t*)ws.g1_first,
          clear ? 2 * (int)pl.sh.n1 : 0, ws.ctr);
    };
    if (pass > 0)
      k_sort_hist<NT><<<blocks, NT, 0, st>>>(KeysInPlace{}, kin, B, sk.sentinel, shift, bits, folds, ws.cnt, nullptr, 0,
                                             ws.ctr);
    else if (sk.low > 0)  // by prefix
      first(PrefixSource{src, sk.low, pl.user_n1, pl.sh.n2, pl.sh.n3});
    else
      first(src);
  } else {
    auto scatter = [&](auto kernel, auto ops) { kernel<<<blocks, NT, 0, st>>>(ops, B, bits, ws.cnt, ws.tot); };
    if (pass == 0) {
      SortOps<true> ops{kin, nullptr, kout, vout, shift, (1u << bits) - 1u};
      folds ? scatter(k_sort_scatter<NT, true, true>, ops) : scatter(k_sort_scatter<NT, true, false>, ops);
    } else {
      SortOps<false> ops{kin, vin, kout, vout, shift, (1u << bits) - 1u};
      folds ? scatter(k_sort_scatter<NT, false, true>, ops) : scatter(k_sort_scatter<NT, false, false>, ops);
    }
  }
}

void launch_sort_pass(const Plan& pl, const Workspace& ws, const SortKeys& sk, const IdSource& src, int B,
                      int pass, bool beside, bool clear, hipStream_t st,
                      int which /*0 = histogram, 1 = scatter, 2 = column scan*/) {
  switch (sort_threads(B, beside)) {
    case 256: sort_pass<256>(pl, ws, sk, src, B, pass, beside, clear, st, which); break;
    case 512: sort_pass<512>(pl, ws, sk, src, B, pass, beside, clear, st, which); break;
    default: sort_pass<1024>(pl, ws, sk, src, B, pass, beside, clear, st, which); break;
  }
}

// The segment kernels of a batch of B items: 1024 threads with 1, 2 or 4 slots each.
template <class F>
static void with_slot_items(const Plan& pl, int B, bool beside, F&& launch) {
  const int span = slot_span(pl.sh, B, beside), blocks = cdiv(B, span);
  if (span == kSegThreads) launch(std::integral_constant<int, 1>{}, blocks);
  else if (span == 2 * kSegThreads) launch(std::integral_constant<int, 2>{}, blocks);
  else launch(std::integral_constant<int, 4>{}, blocks);
}

void launch_seg_count(const Plan& pl, const Workspace& ws, int B, bool beside, hipStream_t st) {
  with_slot_items(pl, B, beside, [&](auto items, int blocks) {
    k_seg_count<items()><<<blocks, kSegThreads, 0, st>>>(ws.key[pl.keys.sorted()], B, pl.sh.N, pl.sh.n3,
                                                         ws.seg_nu, ws.seg_nq);
  });
}

void launch_seg_write(const Plan& pl, const Workspace& ws, int B, bool beside, hipStream_t st) {
  const int f = pl.keys.sorted(), p3 = up8(pl.sh.n3), p2 = up8(pl.sh.n2);
  with_slot_items(pl, B, beside, [&](auto items, int blocks) {
    k_seg_write<items()><<<blocks, kSegThreads, (p3 + p2) * 4, st>>>(
        ws.key[f], ws.val[f], B, pl.sh, p3, p2, ws.seg_nu, ws.seg_nq, ws.s_u, ws.s_rec, ws.u_rs, ws.u_i3, ws.u_q,
        ws.u_code, ws.q_us, ws.q_i1, ws.q_i2, ws.seg_base, ws.seg_rows, ws.g1_first, ws.g1_end, ws.ctr);
  });
}

// prefixes_only: prefixes by i2, all a lookup needs, and not the unique ids by i3
void launch_group(const Plan& pl, const Workspace& ws, int B, bool beside, bool prefixes_only, hipStream_t st) {
  const int span = slot_span(pl.sh, B, beside), nblk = cdiv(B, span), ub = prefixes_only ? 0 : nblk + 1;
  const int p3 = up8(pl.sh.n3), p2 = up8(pl.sh.n2);
  auto launch = [&](auto kernel, int threads) {
    kernel<<<ub + nblk, threads, group_lds(threads, std::max(p3, p2)), st>>>(
        pl.sh, ub, nblk, chunk3_fill(B), p3, p2, ws.seg_base, ws.seg_rows, ws.u_i3, ws.u_code, ws.u_q, ws.q_i2,
        ws.q_i1, ws.q_us, ws.c3_start, ws.c3_desc, ws.c3_item, ws.c2_start, ws.c2_desc, ws.c2_item,
        ws.walk3, ws.ctr);
  };
  switch (span) {
    case 1024: launch(k_group<256>, 256); break;
    case 2048: launch(k_group<512>, 512); break;
    default: launch(k_group<1024>, 1024);
  }
}

}  // namespace ttemb
