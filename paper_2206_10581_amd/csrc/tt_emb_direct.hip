// Kernels that need no index structures (gfx950, fp32).
//
// Small batches.  Sorting and grouping a few thousand ids costs a dozen dependent launches of 3 to
// 10 us each, far more than the arithmetic it saves, so a small batch treats every item (a batch
// position, or a slab of one) as an id and a prefix of its own and takes three launches in all:
//   k_direct_fwd     per item: P = G1[i1] G2[i2], E = P G3[i3], row stored; P kept for backward
//   k_direct_bwd     per item: dP = g G3[i3]^T, its terms of dG3[i3] = P^T g and
//                    dG1[i1] = dP G2[i2]^T, and a copy of the G1 slice (the next kernel overwrites it)
//   k_direct_apply   per slice: finds the items that touch it by scanning the batch's digits, adds
//                    up their terms (for G2: G1^T dP, a contraction over the items) in batch order
//                    and applies the update rule
// Every sum runs over the items in batch order, dealt to a fixed number of threads: results are
// reproducible bit for bit.
//
// Table rows.  k_table_* write a run of consecutive rows of the dense table: all n3 rows of a prefix
// share its product, and no id has to be looked at.
#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "tt_emb_internal.h"

namespace ttemb {

constexpr int kDThreads = 256;
constexpr int kDWaves = kDThreads / kWave;
constexpr int kDirectMax = 8192;             // most items of a batch on these kernels
constexpr size_t kDirectLds = 64 * 1024;     // dynamic LDS of a block of the per-item kernels

// Columns of P = A Bm by a team of TEAM threads: A = d1 x r1 (wavefront-uniform address: scalar
// loads), Bm = r1 x W row-major.  A thread owns VEC neighbouring columns at a time and four rows;
// KU rows of Bm are in flight together.  put(row j1, column, value) takes the results.
template <int TEAM, int VEC, class PUT>
__device__ __forceinline__ void prefix_columns(int t, int d1, int r1, int W, const float* __restrict__ A,
                                               const float* __restrict__ Bm, PUT put) {
  constexpr int KU = 16;
  for (int j0 = 0; j0 < d1; j0 += 4) {
    const float* arow[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) arow[x] = A + (size_t)min(j0 + x, d1 - 1) * r1;
    for (int c = t * VEC; c < W; c += TEAM * VEC) {
      float acc[4][VEC];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[x][v] = 0.f;
      const float* bp = Bm + c;
      int k = 0;
      for (; k + KU <= r1; k += KU) {
        float b[KU][VEC];
#pragma unroll
        for (int j = 0; j < KU; ++j)
#pragma unroll
          for (int v = 0; v < VEC; ++v) b[j][v] = bp[(size_t)(k + j) * W + v];
        __builtin_amdgcn_sched_barrier(0);  // the loads of a round are in flight together
#pragma unroll
        for (int j = 0; j < KU; ++j)
#pragma unroll
          for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[x][v] = fmaf(arow[x][k + j], b[j][v], acc[x][v]);
      }
      if (k < r1) {  // the last, shorter round: rows past r1 read the last one and count zero, in
                     // both operands (zero times an infinity would not be zero)
        float b[KU][VEC];
#pragma unroll
        for (int j = 0; j < KU; ++j)
#pragma unroll
          for (int v = 0; v < VEC; ++v) b[j][v] = bp[(size_t)min(k + j, r1 - 1) * W + v];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < KU; ++j)
#pragma unroll
          for (int v = 0; v < VEC; ++v) b[j][v] = k + j < r1 ? b[j][v] : 0.f;
#pragma unroll
        for (int j = 0; j < KU; ++j)
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const float a = k + j < r1 ? arow[x][min(k + j, r1 - 1)] : 0.f;
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[x][v] = fmaf(a, b[j][v], acc[x][v]);
          }
      }
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (j0 + x < d1)
#pragma unroll
          for (int v = 0; v < VEC; ++v) put(j0 + x, c + v, acc[x][v]);
    }
  }
}

// n floats of global memory, NR per thread in flight at once; fetch starts the loads, put stores
// them to LDS (and moves what does not fit NR registers per thread).
template <int TEAM, int NR>
struct Staged {
  float v[NR];
  __device__ __forceinline__ void fetch(const float* __restrict__ src, int n, int t) {
#pragma unroll
    for (int i = 0; i < NR; ++i) v[i] = src[min(t + i * TEAM, n - 1)];
  }
  template <class PUT>
  __device__ __forceinline__ void put(const float* __restrict__ src, int n, int t, PUT dst) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (t + i * TEAM < n) dst(t + i * TEAM, v[i]);
    for (int i = t + NR * TEAM; i < n; i += TEAM) dst(i, src[i]);
  }
};

template <int TW>
__device__ __forceinline__ void team_sync() {
  if constexpr (TW == 1) wave_sync();
  else __syncthreads();
}

// LDS floats of a team in the forward and the backward kernel (each part a multiple of four)
static inline int up4(int n) { return (n + 3) & ~3; }
static inline int fwd_lds_floats(const Shape& s) { return up4(s.S3) + up4(s.M * (s.r2 + 1)); }
static inline int bwd_lds_floats(const Shape& s, int team) {
  return up4(s.D) + up4(s.S3) + up4(s.M * (s.r2 + 1)) + up4(s.PN) + 4 * team;
}

// ---------------------------------------------------------------------------------------------
// One item per team of TW wavefronts (one for unfolded G2 slices of up to 128 columns, else four).
// Bound by latency: ids, then the slices (one round trip, all of an item's loads side by side), then
// the store.  Measured at 1025 ids, n = 136^3, rank 32: the whole lookup takes one launch of 6 us
// where the sorted path takes nine launches and 55 us.
template <int TW, int VEC, bool TRAIN>
__global__ __launch_bounds__(kDThreads) void k_direct_fwd(
    Shape sh, IdSource src, int B, const float* __restrict__ g1, const float* __restrict__ g2,
    const float* __restrict__ g3, uint32_t* __restrict__ keys, uint16_t* __restrict__ dig, int stride,
    float* __restrict__ P, float* __restrict__ out) {
  constexpr int TEAM = TW * kWave, TPB = kDThreads / TEAM;
  extern __shared__ __align__(16) float lds[];
  const int team = TW == 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave) : 0;
  const int t = threadIdx.x % TEAM;
  const int e = blockIdx.x * TPB + team;
  if (e >= B) return;  // whole teams only, and a block is one team where it has barriers
  const int ps = sh.r2 + 1;
  float* cl = lds + (size_t)team * (((sh.S3 + 3) & ~3) + ((sh.M * ps + 3) & ~3));
  float* pl = cl + ((sh.S3 + 3) & ~3);
  const uint32_t key = (uint32_t)__builtin_amdgcn_readfirstlane((int)key_of_id(src, e, sh.N));
  const bool valid = key < sh.N;
  const uint32_t q = key / sh.n3, i3 = key - q * sh.n3, i1 = q / sh.n2, i2 = q - i1 * sh.n2;
  if (t == 0 && keys != nullptr) keys[e] = key;
  if (TRAIN && t == 0) {
    dig[e] = valid ? (uint16_t)i1 : 0xffffu;
    dig[stride + e] = valid ? (uint16_t)i2 : 0xffffu;
    dig[2 * stride + e] = valid ? (uint16_t)i3 : 0xffffu;
  }
  float* o = out + (size_t)e * sh.D;
  if (!valid) {
    for (int i = t; i < sh.D; i += TEAM) o[i] = 0.f;
    return;
  }
  const float* C = g3 + (size_t)i3 * sh.S3;
  Staged<TEAM, 4> c;
  c.fetch(C, sh.S3, t);
  float* Pe = TRAIN ? P + (size_t)e * sh.PN : nullptr;
  prefix_columns<TEAM, VEC>(t, sh.d1, sh.r1, sh.W, g1 + (size_t)i1 * sh.S1, g2 + (size_t)i2 * sh.S2,
                            [&](int j1, int col, float v) {
                              const int j2 = col / sh.r2;
                              pl[(j1 * sh.d2 + j2) * ps + col - j2 * sh.r2] = v;
                              if (TRAIN) Pe[(size_t)j1 * sh.W + col] = v;
                            });
  c.put(C, sh.S3, t, [&](int i, float v) { cl[i] = v; });
  team_sync<TW>();
  for (int i = t; i < sh.D; i += TEAM) {
    const int m = i / sh.d3, j3 = i - m * sh.d3;
    const float *pr = pl + m * ps, *cc = cl + j3;
    float acc = 0.f;
#pragma unroll 8
    for (int k = 0; k < sh.r2; ++k) acc = fmaf(pr[k], cc[k * sh.d3], acc);
    o[i] = acc;
  }
}

// Lists the parts beyond the first of the slices of one core that more than `most` items share, and
// clears the tickets of those parts; for a whole block, with `bins` words of LDS.  (Counted per item with
// device atomics, 8192 items of three cores took 56 us.)
__device__ void list_hot_parts(uint32_t* lds, int bins, const uint16_t* __restrict__ dig, int B, int n,
                               int most, int2* __restrict__ hot, uint32_t* __restrict__ n_hot, uint32_t* __restrict__ tickets,
                               int n_tickets) {
  const int tid = threadIdx.x;
  uint32_t* listed = lds;  // one word, then the counters
  uint32_t* cnt = lds + 1;
  bins -= 1;
  for (int i = tid; i < n_tickets; i += kDThreads) tickets[i] = 0u;
  if (tid == 0) *listed = 0u;
  for (int s0 = 0; s0 < n; s0 += bins) {
    const int here = min(bins, n - s0);
    for (int i = tid; i < here; i += kDThreads) cnt[i] = 0u;
    __syncthreads();
    constexpr int kLoads = kDirectMax / (kDThreads * 8);
    uint4 d[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int at = (k * kDThreads + tid) * 8;
      d[k] = at < B ? *(const uint4*)(dig + at) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const uint32_t v[4] = {d[k].x, d[k].y, d[k].z, d[k].w};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // 0xffff, an out-of-range id, is past every slice
        const int s = (int)(j % 2 ? v[j / 2] >> 16 : v[j / 2] & 0xffffu) - s0;
        if ((k * kDThreads + tid) * 8 + j < B && s >= 0 && s < here) atomicAdd(&cnt[s], 1u);
      }
    }
    __syncthreads();
    for (int i = tid; i < here; i += kDThreads)
      for (int p = 1; p * most < (int)cnt[i]; ++p) hot[atomicAdd(listed, 1u)] = make_int2(s0 + i, p);
    __syncthreads();
  }
  if (tid == 0) *n_hot = *listed;
}

template <int TW>
__global__ __launch_bounds__(kDThreads) void k_direct_bwd(
    Shape sh, int B, const uint32_t* __restrict__ keys, const float* __restrict__ g1,
    const float* __restrict__ g2, const float* __restrict__ g3, const float* __restrict__ grad,
    const float* __restrict__ P, float* __restrict__ dP, float* __restrict__ g1c,
    float* __restrict__ dg1, float* __restrict__ dg3, const uint16_t* __restrict__ dig, int stride,
    int lds_words, int max_hot, int hot_pieces, int2* __restrict__ hot, uint32_t* __restrict__ n_hot) {
  constexpr int TEAM = TW * kWave, TPB = kDThreads / TEAM;
  extern __shared__ __align__(16) float lds[];
  const int listing = max_hot > 0 ? 3 : 0;  // blocks in front, one per core
  if ((int)blockIdx.x < listing) {
    const int core = blockIdx.x;
    list_hot_parts((uint32_t*)lds, lds_words, dig + core * stride, B,
                   (int)(core == 0 ? sh.n1 : core == 1 ? sh.n2 : sh.n3), direct_part(sh), hot + core * max_hot, n_hot + core,
                   n_hot + 3 + core * max_hot * hot_pieces, max_hot * hot_pieces);
    return;
  }
  const int team = TW == 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave) : 0;
  const int t = threadIdx.x % TEAM;
  const int e = ((int)blockIdx.x - listing) * TPB + team;
  if (e >= B) return;
  const uint32_t key = (uint32_t)__builtin_amdgcn_readfirstlane((int)keys[e]);
  if (key >= sh.N) return;  // no digit row names this item: nothing of it is ever read
  const uint32_t q = key / sh.n3, i3 = key - q * sh.n3, i1 = q / sh.n2, i2 = q - i1 * sh.n2;
  const int ps = sh.r2 + 1;
  const int nD = (sh.D + 3) & ~3, nC = (sh.S3 + 3) & ~3, nP = (sh.M * ps + 3) & ~3,
            nd = (sh.PN + 3) & ~3;
  float* gl = lds + (size_t)team * (nD + nC + nP + nd + 4 * TEAM);
  float* cl = gl + nD;
  float* pl = cl + nC;
  float* dl = pl + nP;
  float* red = dl + nd;
  const float *G = grad + (size_t)e * sh.D, *C = g3 + (size_t)i3 * sh.S3, *Pe = P + (size_t)e * sh.PN;
  const float* A = g1 + (size_t)i1 * sh.S1;
  {
    Staged<TEAM, 4> g, c;
    Staged<TEAM, 8> p;
    Staged<TEAM, 2> a;
    g.fetch(G, sh.D, t);
    c.fetch(C, sh.S3, t);
    p.fetch(Pe, sh.PN, t);
    a.fetch(A, sh.S1, t);
    __builtin_amdgcn_sched_barrier(0);
    g.put(G, sh.D, t, [&](int i, float v) { gl[i] = v; });
    c.put(C, sh.S3, t, [&](int i, float v) { cl[i] = v; });
    p.put(Pe, sh.PN, t, [&](int i, float v) { pl[(i / sh.r2) * ps + i % sh.r2] = v; });
    float* Ac = g1c + (size_t)e * sh.S1;
    a.put(A, sh.S1, t, [&](int i, float v) { Ac[i] = v; });
  }
  team_sync<TW>();
  // dP[m][b] = sum over j3 of g[m][j3] G3[b][j3]
  float* de = dP + (size_t)e * sh.PN;
  for (int i = t; i < sh.PN; i += TEAM) {
    const int m = i / sh.r2, b = i - m * sh.r2;
    float acc = 0.f;
    for (int j = 0; j < sh.d3; ++j) acc = fmaf(gl[m * sh.d3 + j], cl[b * sh.d3 + j], acc);
    dl[i] = acc;
    de[i] = acc;
  }
  // term of dG3: sum over m of P[m][b] g[m][j3]
  float* w3 = dg3 + (size_t)e * sh.S3;
  for (int i = t; i < sh.S3; i += TEAM) {
    const int b = i / sh.d3, j = i - b * sh.d3;
    float acc = 0.f;
    for (int m = 0; m < sh.M; ++m) acc = fmaf(pl[m * ps + b], gl[m * sh.d3 + j], acc);
    w3[i] = acc;
  }
  team_sync<TW>();
  // term of dG1: dP[j1][c] G2[i2][a][c] summed over the W columns c.  Thread (part, a) walks a share
  // of the columns of row a, four at a time where rows are 16-byte aligned.
  const float* Bm = g2 + (size_t)i2 * sh.S2;
  float* w1 = dg1 + (size_t)e * sh.S1;
  for (int a0 = 0; a0 < sh.r1; a0 += TEAM) {
    const int ra = min(TEAM, sh.r1 - a0);
    const int parts = TEAM / ra, part = t / ra;
    const int a = a0 + t % ra;
    const bool on = part < parts;
    const int quads = (sh.W + 3) / 4, per = (quads + parts - 1) / parts;
    const int c0 = on ? min(part * per * 4, sh.W) : 0, c1 = on ? min(c0 + per * 4, sh.W) : 0;
    const float* row = Bm + (size_t)a * sh.W;
    for (int j0 = 0; j0 < sh.d1; j0 += 4) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      const float* dr[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) dr[x] = dl + min(j0 + x, sh.d1 - 1) * sh.W;
      if (sh.W % 4 == 0) {
        int c = c0;
        for (; c + 32 <= c1; c += 32) {
          f4 b[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) b[j] = *(const f4*)(row + c + 4 * j);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const f4 d = *(const f4*)(dr[x] + c + 4 * j);
              acc[x] = fmaf(d.x, b[j].x, acc[x]);
              acc[x] = fmaf(d.y, b[j].y, acc[x]);
              acc[x] = fmaf(d.z, b[j].z, acc[x]);
              acc[x] = fmaf(d.w, b[j].w, acc[x]);
            }
        }
        for (; c < c1; c += 4) {
          const f4 b = *(const f4*)(row + c);
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const f4 d = *(const f4*)(dr[x] + c);
            acc[x] = fmaf(d.x, b.x, acc[x]);
            acc[x] = fmaf(d.y, b.y, acc[x]);
            acc[x] = fmaf(d.z, b.z, acc[x]);
            acc[x] = fmaf(d.w, b.w, acc[x]);
          }
        }
      } else {
        for (int c = c0; c < c1; ++c) {
          const float b = row[c];
#pragma unroll
          for (int x = 0; x < 4; ++x) acc[x] = fmaf(dr[x][c], b, acc[x]);
        }
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) red[x * TEAM + t] = acc[x];
      team_sync<TW>();
      for (int i = t; i < 4 * ra; i += TEAM) {
        const int x = i / ra, aa = i - x * ra;
        if (j0 + x < sh.d1) {
          float s = 0.f;
          for (int p = 0; p < parts; ++p) s += red[x * TEAM + p * ra + aa];
          w1[(size_t)(j0 + x) * sh.r1 + a0 + aa] = s;
        }
      }
      team_sync<TW>();
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Sums and update.  A block owns a run of entries of one slice:
//   G2 jobs (first, they are the longest): 16*RT rows and 16*CT columns of the slice, as sum over
//     items of G1^T (r1 x d1) dP (d1 x W), one 16x16x4 matrix-core product per item, four rows of
//     d1 and tile (edges masked), the items dealt to the four wavefronts.  (512 ids of d = (5,3,4) at
//     rank 16: 20 us a step, 45 with one id in all positions, where a vector-ALU form for d1 > 4
//     without loads in flight took 30 and 333; the indexed kernels 97 and 77.)
//   G3, then G1 jobs: up to 256*VEC entries, the items dealt to groups of threads
// Such a block takes the first direct_part() items of its slice.  One compute unit fetches some 20 items a
// microsecond, so a slice that more items share (a hot id, neighbouring ids) is cut into parts: the
// backward kernel lists those beyond the first, blocks at the front of the grid take them, and the block
// of a slice's piece that ends last adds the parts up in order and updates.  8192 ids at rank 16 of
// n = 136^3, one step, in one block -> in parts of 512 (the indexed kernels): one id 397 -> 67 us (79),
// 200 neighbouring ids 284 -> 66 (131), Zipf 1.2 87 -> 64 (91), uniform 41 -> 42 (98).  Parts of 256 are
// a few us faster there, but cut slices that one block adds up sooner: n = (40,30,20), d = (5,3,4),
// uniform ids 58 -> 72 us.
// Sums have two levels, a short chain of the items that are in flight together and a chain of those
// rounds, and groups join in pairs.  Error of dG2 for 1024 copies of one id (terms of one sign, 2-norm):
// 6.5e-8, as on the indexed kernels, where one chain over all of a wavefront's items left 2.5e-7;
// dG3 of the smallest slices, 128 groups, 6e-8, where joining them in a chain left 2.1e-7.
struct DirectList {
  uint16_t item[kDirectMax];
  uint32_t wave_n[kDWaves];
};

__device__ __forceinline__ int direct_list(DirectList& L, const uint16_t* __restrict__ dig, int B, int want) {
  constexpr int kStep = kWave * 8, kMaxSteps = kDirectMax / (kDWaves * kStep);
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int steps = (B + kDWaves * kStep - 1) / (kDWaves * kStep);  // at most kMaxSteps
  const int base = w * steps * kStep;
  uint4 d[kMaxSteps];
#pragma unroll
  for (int s = 0; s < kMaxSteps; ++s) {
    const int at = base + s * kStep + lane * 8;
    d[s] = (s < steps && at < B) ? *(const uint4*)(dig + at) : make_uint4(~0u, ~0u, ~0u, ~0u);
  }
  uint32_t mask[kMaxSteps], incl[kMaxSteps], n = 0;
#pragma unroll
  for (int s = 0; s < kMaxSteps; ++s) {
    const int at = base + s * kStep + lane * 8;
    const uint32_t v[4] = {d[s].x, d[s].y, d[s].z, d[s].w};
    uint32_t m = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if ((v[j] & 0xffffu) == (uint32_t)want) m |= 1u << (2 * j);
      if ((v[j] >> 16) == (uint32_t)want) m |= 2u << (2 * j);
    }
    if (s >= steps || at >= B) m = 0;
    else if (at + 8 > B) m &= (1u << (B - at)) - 1u;  // digits past the batch are unwritten
    mask[s] = m;
    incl[s] = n + wave_inclusive_scan((uint32_t)__popc(m), lane);
    n = (uint32_t)__builtin_amdgcn_readlane((int)incl[s], kWave - 1);
  }
  if (lane == 0) L.wave_n[w] = n;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int k = 0; k < kDWaves; ++k) {
    before += k < w ? L.wave_n[k] : 0u;
    total += L.wave_n[k];
  }
#pragma unroll
  for (int s = 0; s < kMaxSteps; ++s) {
    uint32_t at = before + incl[s] - (uint32_t)__popc(mask[s]);
    for (uint32_t m = mask[s]; m != 0; m &= m - 1)
      L.item[at++] = (uint16_t)(base + s * kStep + lane * 8 + __ffs((int)m) - 1);
  }
  __syncthreads();
  return (int)total;
}

// Blocks that stand for the slices of a core: one per slice, or, where the batch has fewer items than the
// core has slices, one per item, which takes the slice if no earlier item shares it.  A batch never
// launches more than its items can fill: a single id at n = (60000,20,20) takes 18 us instead of 65
// (the indexed kernels: 119), and no grid grows with the table.
__host__ __device__ inline int slice_blocks(uint32_t n, int B) { return B < (int)n ? B : (int)n; }

// Pairwise sums of what `groups` groups (a power of two) of `lanes` threads hold, left in the first group.
template <int VEC>
__device__ __forceinline__ void join_groups(float* red, int tid, int lanes, int groups, float* acc) {
  for (int half = groups / 2; half > 0; half /= 2) {
    if (tid >= half * lanes && tid < 2 * half * lanes)
#pragma unroll
      for (int x = 0; x < VEC; ++x) red[tid * VEC + x] = acc[x];
    __syncthreads();
    if (tid < half * lanes)
#pragma unroll
      for (int x = 0; x < VEC; ++x) acc[x] += red[(tid + half * lanes) * VEC + x];
  }
}

// What a block of a slice cut into parts needs to find its siblings; for a whole block.
struct DirectParts {
  int slot[kDirectMax / kDirectPartLeast];  // part -> its place among the listed parts of all cores
  uint32_t last;
};
// Leaves in P where the sums of this slice's parts lie.
__device__ __forceinline__ void find_parts(DirectParts& P, const int2* __restrict__ hot, int first, int n_hot,
                                           int slice) {
  for (int i = threadIdx.x; i < n_hot; i += kDThreads) {
    const int2 h = hot[first + i];
    if (h.x == slice) P.slot[h.y] = first + i;
  }
  __syncthreads();
}
// Sums of a part go past the L2 of this block's XCD and are read past the reader's: stores and loads at
// agent scope.  A store that has completed (s_waitcnt) is therefore visible to every block, and no cache
// has to be written back or invalidated (fences that do took 5 to 10 us per part).
__device__ __forceinline__ void put_sum(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float get_sum(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// True in the block that is the last of `parts` to come here with this ticket: all parts' sums are
// there.
__device__ __forceinline__ bool last_part(DirectParts& P, uint32_t* ticket, int parts) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's sums are stored
  __syncthreads();                                  // and those of the others of the block
  if (threadIdx.x == 0)
    P.last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == (uint32_t)parts;
  __syncthreads();
  return P.last != 0;
}

// PARTS: slices of more than direct_part() items are cut into parts (the batch has that many)
template <int RT, int CT, int RULE, bool PARTS>
__global__ __launch_bounds__(kDThreads) void k_direct_apply(
    Shape sh, int B, float lr, UpdateRule ada, const uint16_t* __restrict__ dig, int stride,
    const float* __restrict__ g1c, const float* __restrict__ dP, const float* __restrict__ dg1,
    const float* __restrict__ dg3, uint32_t* n_hot, const int2* __restrict__ hot, int max_hot, int hot_pieces,
    float* hot_sum, float* __restrict__ g1, float* __restrict__ g2,
    float* __restrict__ g3) {
  constexpr bool ADA = RULE != kUpdateSgd, ADAM = RULE == kUpdateAdam;
  constexpr int kRed = std::max(kDWaves * RT * CT * 256, kDThreads * 4);
  __shared__ DirectList L;
  __shared__ float red[kRed];
  const int tid = threadIdx.x;
  __shared__ DirectParts parts_of;
  const int cols2 = (sh.W + 16 * CT - 1) / (16 * CT), per2 = cols2 * ((sh.r1 + 16 * RT - 1) / (16 * RT));
  const int per3 = (sh.S3 + 1023) / 1024, per1 = (sh.S1 + 1023) / 1024;
  const int most_s = max(max(sh.S1, sh.S2), sh.S3);
  // core (0, 1, 2 for G1, G2, G3), slice, piece of the slice and part of its items
  int core, slice, piece, part = 0;
  int first = -1;  // a block that stands for an item: the item, which has to be its slice's first
  int job = blockIdx.x;
  const int hot_jobs = PARTS ? 3 * max_hot * hot_pieces : 0;  // blocks of parts beyond the first
  if (PARTS && job < hot_jobs) {
    const int listed = job / hot_pieces;
    core = listed / max_hot, piece = job % hot_pieces;
    if (listed - core * max_hot >= (int)n_hot[core]) return;
    slice = hot[listed].x, part = hot[listed].y;
    if (piece >= (core == 0 ? per1 : core == 1 ? per2 : per3)) return;
  } else {
    job -= hot_jobs;
    const int jobs2 = slice_blocks(sh.n2, B) * per2, jobs3 = slice_blocks(sh.n3, B) * per3;
    core = job < jobs2 ? 1 : job < jobs2 + jobs3 ? 2 : 0;
    job -= core == 1 ? 0 : core == 2 ? jobs2 : jobs2 + jobs3;
    const int per = core == 1 ? per2 : core == 2 ? per3 : per1;
    piece = job % per;
    slice = job / per;
    if (B < (int)(core == 1 ? sh.n2 : core == 2 ? sh.n3 : sh.n1)) {
      first = slice;
      slice = (int)dig[core * stride + first];
      if (slice == 0xffff) return;  // an out-of-range id
    }
  }
  int n = direct_list(L, dig + core * stride, B, slice);
  if (first >= 0 && (int)L.item[0] != first) return;
  n = __builtin_amdgcn_readfirstlane(n);  // the same in all threads
  const int most = direct_part(sh), parts = PARTS && n > most ? (n + most - 1) / most : 1;
  const int lo = PARTS ? part * most : 0, hi = parts > 1 ? min(n, lo + most) : n;
  if (lo >= hi) return;
  const int S = core == 0 ? sh.S1 : core == 1 ? sh.S2 : sh.S3;
  float* G = (core == 0 ? g1 : core == 1 ? g2 : g3) + (size_t)slice * S;
  float* St = ADA ? (core == 0 ? ada.s1 : core == 1 ? ada.s2 : ada.s3) + (size_t)slice * S : nullptr;
  float* Vt = ADAM ? (core == 0 ? ada.v1 : core == 1 ? ada.v2 : ada.v3) + (size_t)slice * S : nullptr;
  if (PARTS && parts > 1) find_parts(parts_of, hot, core * max_hot, (int)n_hot[core], slice);
  // where part p leaves its sums; entries are taken or summed up by the thread that owns them
  auto sums_of = [&](int p) {
    return hot_sum + (size_t)(p > 0 ? parts_of.slot[p] : 3 * max_hot + parts_of.slot[1]) * most_s;
  };
  auto update = [&](size_t at, float old, float s) {
    G[at] = updated_entry<RULE>(old, s, lr, ada, ADA ? St + at : nullptr, ADAM ? Vt + at : nullptr);
  };
  auto put = [&](size_t at, float old, float s) {
    if (!PARTS || parts == 1) update(at, old, s);
    else put_sum(sums_of(part) + at, s);
  };
  auto update_from_parts = [&](size_t at) {
    float s = get_sum(sums_of(0) + at);
    for (int p = 1; p < parts; ++p) s += get_sum(sums_of(p) + at);
    update(at, G[at], s);
  };
  auto is_last = [&] {
    return PARTS && parts > 1 &&
           last_part(parts_of, &n_hot[3 + parts_of.slot[1] * hot_pieces + piece], parts);
  };
  if (core == 1) {
    constexpr int U = RT >= 4 ? 4 : 8;  // items in flight per wavefront
    const int w = tid / kWave, lane = tid % kWave, l16 = lane % 16, kg = lane / 16;
    const int col0 = piece % cols2 * 16 * CT, row0 = piece / cols2 * 16 * RT;
    // rows and columns past the slice read a valid address and are not stored; rows past d1 count
    // zero in both operands (zero times an infinity would not be zero)
    int ra[RT], cb[CT];
#pragma unroll
    for (int i = 0; i < RT; ++i) ra[i] = min(row0 + 16 * i + l16, sh.r1 - 1);
#pragma unroll
    for (int j = 0; j < CT; ++j) cb[j] = min(col0 + 16 * j + l16, sh.W - 1);
    constexpr int kOut = RT * CT * 256;
    auto each_entry = [&](auto body) {
#pragma unroll
      for (int x = 0; x < kOut / kDThreads; ++x) {
        const int o = tid + x * kDThreads, row = row0 + o / (16 * CT), col = col0 + o % (16 * CT);
        if (row < sh.r1 && col < sh.W) body(x, o, (size_t)row * sh.W + col);
      }
    };
    // The entries as they are, all at once: read before the first is written.  (With the eight row tiles of
    // rank 128 their registers cost a block per compute unit: 250 ids 69 -> 76 us a step.)
    constexpr bool kAhead = RT < 8;
    float old[kAhead ? kOut / kDThreads : 1];
    if constexpr (kAhead) each_entry([&](int x, int, size_t at) { old[x] = G[at]; });
    f4 sum[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) sum[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    for (int k = lo + w; k < hi; k += kDWaves * U)
      for (int j0 = 0; j0 < sh.d1; j0 += 4) {
        const int j1 = min(j0 + kg, sh.d1 - 1);
        const bool on = j0 + kg < sh.d1;
        float a[U][RT], b[U][CT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e = L.item[min(k + u * kDWaves, hi - 1)];
          const float* ap = g1c + (size_t)e * sh.S1 + j1 * sh.r1;
          const float* bp = dP + (size_t)e * sh.PN + j1 * sh.W;
#pragma unroll
          for (int i = 0; i < RT; ++i) a[u][i] = ap[ra[i]];
#pragma unroll
          for (int j = 0; j < CT; ++j) b[u][j] = bp[cb[j]];
        }
        __builtin_amdgcn_sched_barrier(0);
        f4 acc[RT][CT];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < CT; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (k + u * kDWaves < hi)  // wavefront-uniform
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
              for (int j = 0; j < CT; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(on ? a[u][i] : 0.f, on ? b[u][j] : 0.f,
                                                                 acc[i][j], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < CT; ++j) sum[i][j] += acc[i][j];
      }
    // element v of lane (kg, l16) is row 16*i + 4*kg + v, column 16*j + l16
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          red[((w * RT * 16 + 16 * i + 4 * kg + v) * CT + j) * 16 + l16] = sum[i][j][v];
    __syncthreads();
    each_entry([&](int x, int o, size_t at) {
      float s = red[o];
#pragma unroll
      for (int p = 1; p < kDWaves; ++p) s += red[p * kOut + o];
      put(at, kAhead ? old[kAhead ? x : 0] : G[at], s);
    });
    if (is_last()) each_entry([&](int, int, size_t at) { update_from_parts(at); });
    return;
  }
  const int o0 = piece * 1024, outs = min(1024, S - o0);
  const float* src = (core == 2 ? dg3 : dg1) + o0;
  auto sum = [&](auto vec) {
    constexpr int VEC = decltype(vec)::value, U = 8;
    int lanes = 1;
    while (lanes * VEC < outs && lanes < kDThreads) lanes <<= 1;
    const int groups = kDThreads / lanes, lane = tid % lanes, grp = tid / lanes;
    for (int b0 = 0; b0 < outs; b0 += lanes * VEC) {
      const bool on = b0 + lane * VEC < outs;
      const int o = on ? b0 + lane * VEC : 0;
      float acc[VEC];
#pragma unroll
      for (int x = 0; x < VEC; ++x) acc[x] = 0.f;
      int k = lo + grp;
      for (; k + (U - 1) * groups < hi; k += U * groups) {
        float v[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float* p = src + (size_t)L.item[k + u * groups] * S + o;
#pragma unroll
          for (int x = 0; x < VEC; ++x) v[u][x] = p[x];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < VEC; ++x) {
#pragma unroll
          for (int u = 1; u < U; ++u) v[0][x] += v[u][x];
          acc[x] += v[0][x];
        }
      }
      float rest[VEC];
#pragma unroll
      for (int x = 0; x < VEC; ++x) rest[x] = 0.f;
      for (; k < hi; k += groups) {
        const float* p = src + (size_t)L.item[k] * S + o;
#pragma unroll
        for (int x = 0; x < VEC; ++x) rest[x] += p[x];
      }
#pragma unroll
      for (int x = 0; x < VEC; ++x) acc[x] += rest[x];
      join_groups<VEC>(red, tid, lanes, groups, acc);
      if (grp == 0 && on) {
#pragma unroll
        for (int x = 0; x < VEC; ++x) put(o0 + o + x, G[o0 + o + x], acc[x]);
      }
      __syncthreads();
    }
  };
  if (S % 4 == 0) sum(std::integral_constant<int, 4>{});
  else sum(std::integral_constant<int, 1>{});
  if (is_last())
    for (int o = tid; o < outs; o += kDThreads) update_from_parts(o0 + o);
}

// ---------------------------------------------------------------------------------------------
// Consecutive table rows, shapes with d2 = 4, r1 = r2 = R, d3 in {4, 8} and d1 a multiple of four.
// A wavefront owns NP neighbouring prefixes (of one slab of four G1 rows each) and a run of i3: it
// forms their products P (16 x R), keeps them in registers as one matrix-core operand, and streams
// G3 past them; the product is taken transposed, (i3,j3) x (j1,j2), so that the four accumulator
// elements of a lane are neighbours in the row and a wavefront's 16-byte stores cover whole rows.
// Bound by the row stores.
template <int R>
constexpr int table_np() { return R >= 128 ? 1 : R >= 64 ? 2 : 4; }

template <int R, int D3>
__global__ __launch_bounds__(kDThreads) void k_table_mfma(
    int n2, int n3, int ns, int first, int count, int vp0, int nvp, int nseg, int seg_tiles,
    const float* __restrict__ g1, const float* __restrict__ g2, const float* __restrict__ g3,
    float* __restrict__ out) {
  constexpr int W = 4 * R, S1 = 4 * R, S2 = R * W, S3 = R * D3, D = 16 * D3, UPT = 16 / D3, KQ = R / 4;
  constexpr int NP = table_np<R>(), PS = R + 4, VEC = W >= 128 ? 2 : 1;
  __shared__ __align__(16) float pl[kDWaves][16 * PS];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int l16 = lane % 16, kg = lane / 16;
  const int unit = blockIdx.x * kDWaves + w;
  const int group = unit / nseg, seg = unit - group * nseg;
  const int x0 = group * NP;
  if (x0 >= nvp) return;
  const int t0 = seg * seg_tiles, t1 = min(t0 + seg_tiles, (n3 + UPT - 1) / UPT);
  float b[NP][KQ];
  float* orow[NP];
  int row0[NP];      // first row of the prefix, counted from `first`
  bool any = false;
#pragma unroll
  for (int x = 0; x < NP; ++x) {
    const int vp = vp0 + min(x0 + x, nvp - 1);
    const int prefix = vp / ns, h = vp - prefix * ns;
    row0[x] = x0 + x < nvp ? prefix * n3 - first : INT32_MIN / 2;
    orow[x] = out + (ptrdiff_t)(prefix * n3 - first) * ns * D + (size_t)h * D + l16 * D3 + (4 * kg) % D3;
    // rows [row0 + t0*UPT, row0 + t1*UPT) meet [0, count)
    any = any || (row0[x] + t0 * UPT < count && row0[x] + t1 * UPT > 0);
  }
  if (!any) return;
#pragma unroll
  for (int x = 0; x < NP; ++x) {
    const int vp = vp0 + min(x0 + x, nvp - 1);
    const int prefix = vp / ns, h = vp - prefix * ns, i1 = prefix / n2, i2 = prefix - i1 * n2;
    prefix_columns<kWave, VEC>(lane, 4, R, W, g1 + (size_t)(i1 * ns + h) * S1, g2 + (size_t)i2 * S2,
                               [&](int j1, int col, float v) {
                                 pl[w][(j1 * 4 + col / R) * PS + col % R] = v;
                               });
    wave_sync();
#pragma unroll
    for (int j = 0; j < KQ; ++j) b[x][j] = pl[w][l16 * PS + KQ * kg + j];
    wave_sync();
  }
  float a[2][KQ];
  auto fetch = [&](float (&av)[KQ], int t) {
    const float* p = g3 + (size_t)min(t * UPT + l16 / D3, n3 - 1) * S3 + (KQ * kg) * D3 + l16 % D3;
#pragma unroll
    for (int j = 0; j < KQ; ++j) av[j] = p[j * D3];
  };
  auto tile = [&](const float (&av)[KQ], int t) {
    const int i3 = t * UPT + (4 * kg) / D3;
#pragma unroll
    for (int x = 0; x < NP; ++x) {
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < KQ; ++j)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j], b[x][j], acc, 0, 0, 0);
      // lane (kg, l16): rows 4*kg .. 4*kg+3 of the tile = four j3 of one i3, column (j1,j2) = l16
      const int row = row0[x] + i3;
      if (i3 < n3 && row >= 0 && row < count)
        __builtin_nontemporal_store(acc, (f4*)(orow[x] + (size_t)i3 * ns * D));
    }
  };
  fetch(a[0], t0);
  for (int t = t0; t < t1; t += 2) {
    fetch(a[1], t + 1);
    tile(a[0], t);
    if (t + 1 >= t1) break;
    fetch(a[0], t + 2);
    tile(a[1], t + 1);
  }
}

// The same for any shape: a block owns one prefix and a run of i3; P and the G3 slices of kTableIds
// ids at a time sit in LDS, every thread forms outputs of the run's rows in order.
constexpr int kTableIds = 8;

__global__ __launch_bounds__(kDThreads) void k_table_any(Shape sh, int first, int count, int p0, int nseg,
                                                         int seg_ids, const float* __restrict__ g1,
                                                         const float* __restrict__ g2,
                                                         const float* __restrict__ g3,
                                                         float* __restrict__ out) {
  extern __shared__ __align__(16) float lds[];
  const int prefix = p0 + (int)blockIdx.x / nseg, seg = (int)blockIdx.x % nseg;
  const int ps = sh.r2 + 1;
  float* cl = lds;                                  // kTableIds G3 slices
  float* pl = lds + ((kTableIds * sh.S3 + 3) & ~3);
  const int row0 = prefix * (int)sh.n3 - first;     // table rows before `first` are negative
  const int a0 = max(seg * seg_ids, -row0), a1 = min(min((seg + 1) * seg_ids, (int)sh.n3), count - row0);
  if (a0 >= a1) return;
  const int i1 = prefix / (int)sh.n2, i2 = prefix - i1 * (int)sh.n2;
  prefix_columns<kDThreads, 1>((int)threadIdx.x, sh.d1, sh.r1, sh.W, g1 + (size_t)i1 * sh.S1,
                               g2 + (size_t)i2 * sh.S2, [&](int j1, int col, float v) {
                                 const int j2 = col / sh.r2;
                                 pl[(j1 * sh.d2 + j2) * ps + col - j2 * sh.r2] = v;
                               });
  for (int i3 = a0; i3 < a1; i3 += kTableIds) {
    const int ids = min(kTableIds, a1 - i3);
    __syncthreads();
    const float* C = g3 + (size_t)i3 * sh.S3;
    for (int i = threadIdx.x; i < ids * sh.S3; i += kDThreads) cl[i] = C[i];
    __syncthreads();
    float* o = out + (size_t)(row0 + i3) * sh.D;
    for (int i = threadIdx.x; i < ids * sh.D; i += kDThreads) {
      const int id = i / sh.D, e = i - id * sh.D, m = e / sh.d3, j3 = e - m * sh.d3;
      const float *pr = pl + m * ps, *cc = cl + id * sh.S3 + j3;
      float acc = 0.f;
#pragma unroll 8
      for (int k = 0; k < sh.r2; ++k) acc = fmaf(pr[k], cc[k * sh.d3], acc);
      __builtin_nontemporal_store(acc, o + i);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// host side

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

static int team_waves(const Shape& s) { return s.W > 2 * kWave ? 4 : 1; }

// Largest batch (in items) that takes the index-free kernels; 0 for shapes they do not hold.
// Every item reads its whole G2 slice, which the sorted path reads once per sixteen prefixes: past
// kDirectBytes of slices that costs more than the index launches it saves.  And it forms a product of
// its own: the same bound holds for those (d = (8,9,1), r = (2,100), 28 KiB each: a lookup of 2048 ids 38
// us against 61 to 91, of 8192 125 against 63 to 155).  And it waits for its rounds of loads one after
// the other: past kDirectRounds of them the limit falls (d = (20,1,9), r = (70,2), 25 rounds: 8000 ids 70
// us against 51 to 68).  A training step on these
// kernels and on the indexed ones, us, at the largest batches, for uniform ids and for a single one:
//   rank 8, 8192 ids     40 / 95,  63 / 78        rank 64, 1024 ids    48 / 114, 66 / 81
//   rank 16, 8192 ids    42 / 98,  67 / 79        rank 128, 256 ids    70 / 144, 70 / 93
//   rank 32, 4096 ids    45 / 107, 77 / 75        d = (4,5,5) at rank 32, 2048 ids  39 / 141, 72 / 107
// (n = 136^3, d = (4,4,8)).  A lookup takes 7 to 17 us at these sizes, 50 to 80 on the indexed kernels.
int direct_capacity(const Shape& s) {
  constexpr int64_t kDirectBytes = (int64_t)64 << 20;
  constexpr int64_t kDirectRounds = 16;
  const int tw = team_waves(s), teams = kDWaves / tw;
  if (s.n1 >= 0xffffu) return 0;  // digits are 16-bit
  if ((size_t)teams * fwd_lds_floats(s) * 4 > kDirectLds ||
      (size_t)teams * bwd_lds_floats(s, tw * kWave) * 4 > kDirectLds)
    return 0;
  const int64_t rounds = (int64_t)cdiv(s.d1, 4) * cdiv(s.r1, 16) * cdiv(s.W, 2 * tw * kWave);
  return (int)std::min<int64_t>(kDirectMax * kDirectRounds / std::max(rounds, kDirectRounds),
                                kDirectBytes / ((int64_t)std::max(s.S2, s.PN) * 4));
}

// Pieces that k_direct_apply cuts a slice of G2 into, and the most of any core's slice.
static int row_tiles(const Shape& s) { return s.r1 <= 16 ? 1 : s.r1 <= 32 ? 2 : s.r1 <= 64 ? 4 : 8; }
static int col_tiles(const Shape& s) { return row_tiles(s) <= 2 && s.W % 32 == 0 ? 2 : 1; }
static int pieces2(const Shape& s) { return cdiv(s.W, 16 * col_tiles(s)) * cdiv(s.r1, 16 * row_tiles(s)); }
int direct_pieces(const Shape& s) { return std::max({pieces2(s), cdiv(s.S1, 1024), cdiv(s.S3, 1024)}); }

// The same for a batch that backward_update follows, which keeps 4 (2 PN + 2 S1 + S3) bytes per item:
// no more than kDirectKept of them (8192 items at rank 16 of D = 64 keep 24 MiB, 4096 at rank 32 of
// D = 128 24 MiB; products of thousands of floats would take hundreds).
int direct_train_capacity(const Shape& s) {
  constexpr int64_t kDirectKept = (int64_t)32 << 20;
  const int64_t item = 4 * (2 * (int64_t)s.PN + 2 * (int64_t)s.S1 + s.S3) +
                       4 * 6 * (int64_t)std::max({s.S1, s.S2, s.S3}) / direct_part(s);  // and its share of the parts
  return (int)std::min<int64_t>(direct_capacity(s), kDirectKept / item);
}

void launch_direct_fwd(const Plan& pl, const DirectBuffers& d, const IdSource& src, int B,
                       const float* g1, const float* g2, const float* g3, float* out, bool train,
                       hipStream_t st) {
  const Shape& s = pl.sh;
  const int tw = team_waves(s), grid = cdiv(B, kDWaves / tw);
  const size_t lds = (size_t)(kDWaves / tw) * fwd_lds_floats(s) * sizeof(float);
  const bool vec = s.W > tw * kWave && s.r2 % 2 == 0;
#define TT_DF(TW, V, TR)                                                                          \
  k_direct_fwd<TW, V, TR><<<grid, kDThreads, lds, st>>>(s, src, B, g1, g2, g3, d.key, d.dig, d.stride, \
                                                        d.P, out)
  if (tw == 1) {
    if (vec) { if (train) TT_DF(1, 2, true); else TT_DF(1, 2, false); }
    else { if (train) TT_DF(1, 1, true); else TT_DF(1, 1, false); }
  } else {
    if (vec) { if (train) TT_DF(4, 2, true); else TT_DF(4, 2, false); }
    else { if (train) TT_DF(4, 1, true); else TT_DF(4, 1, false); }
  }
#undef TT_DF
}

void launch_direct_bwd(const Plan& pl, const DirectBuffers& d, int B, const float* g1, const float* g2,
                       const float* g3, const float* grad, hipStream_t st) {
  const Shape& s = pl.sh;
  const int tw = team_waves(s), grid = cdiv(B, kDWaves / tw) + (hot_parts(s, B) > 0 ? 3 : 0);
  const size_t lds = (size_t)(kDWaves / tw) * bwd_lds_floats(s, tw * kWave) * sizeof(float);
  if (tw == 1)
    k_direct_bwd<1><<<grid, kDThreads, lds, st>>>(s, B, d.key, g1, g2, g3, grad, d.P, d.dP, d.g1, d.dg1,
                                                  d.dg3, d.dig, d.stride, (int)(lds / 4), hot_parts(s, B),
                                                  direct_pieces(s), d.hot, d.n_hot);
  else
    k_direct_bwd<4><<<grid, kDThreads, lds, st>>>(s, B, d.key, g1, g2, g3, grad, d.P, d.dP, d.g1, d.dg1,
                                                  d.dg3, d.dig, d.stride, (int)(lds / 4), hot_parts(s, B),
                                                  direct_pieces(s), d.hot, d.n_hot);
}

void launch_direct_apply(const Plan& pl, const DirectBuffers& d, int B, float* g1, float* g2, float* g3,
                         float lr, const UpdateRule& ada, hipEvent_t stop, hipStream_t st) {
  const Shape& s = pl.sh;
  const int rt = row_tiles(s), ct = col_tiles(s), per2 = pieces2(s);
  const int max_hot = hot_parts(s, B), hot_pieces = direct_pieces(s);
  // at most B times the pieces of a slice: the bounds on B keep that to about a million blocks
  const int grid = 3 * max_hot * hot_pieces + slice_blocks(s.n2, B) * per2 + slice_blocks(s.n3, B) * cdiv(s.S3, 1024) +
                   slice_blocks(s.n1, B) * cdiv(s.S1, 1024);
#define TT_DA(RT, CT, RULE, PARTS)                                                                 \
  do {                                                                                             \
    auto kernel = k_direct_apply<RT, CT, RULE, PARTS>;                                             \
    if (stop != nullptr)                                                                           \
      hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(kDThreads), 0, st, nullptr, stop, 0, s, B,    \
                            lr, ada, (const uint16_t*)d.dig, d.stride, (const float*)d.g1,         \
                            (const float*)d.dP, (const float*)d.dg1, (const float*)d.dg3, d.n_hot, \
                            (const int2*)d.hot, max_hot, hot_pieces, d.hot_sum, g1, g2, g3);       \
    else                                                                                           \
      kernel<<<grid, kDThreads, 0, st>>>(s, B, lr, ada, d.dig, d.stride, d.g1, d.dP, d.dg1, d.dg3, \
                                         d.n_hot, d.hot, max_hot, hot_pieces, d.hot_sum, g1, g2,   \
                                         g3);                                                      \
  } while (0)
#define TT_DP(RT, CT, RULE)                                                                        \
  do {                                                                                             \
    if (max_hot > 0) TT_DA(RT, CT, RULE, true);                                                    \
    else TT_DA(RT, CT, RULE, false);                                                               \
  } while (0)
#define TT_DR(RT, CT)                                                                              \
  do {                                                                                             \
    if (ada.kind == kUpdateAdam) TT_DP(RT, CT, kUpdateAdam);                                       \
    else if (ada.kind == kUpdateAdagrad) TT_DP(RT, CT, kUpdateAdagrad);                            \
    else TT_DP(RT, CT, kUpdateSgd);                                                                \
  } while (0)
  if (rt == 1) { if (ct == 2) TT_DR(1, 2); else TT_DR(1, 1); }
  else if (rt == 2) { if (ct == 2) TT_DR(2, 2); else TT_DR(2, 1); }
  else if (rt == 4) TT_DR(4, 1);
  else TT_DR(8, 1);
#undef TT_DR
#undef TT_DP
#undef TT_DA
}

// Whether a run of `count` rows is streamed by these kernels; else the caller looks the rows up.  The
// product and kTableIds G3 slices have to fit a block's LDS.  And every wavefront or block forms its
// prefixes' products by itself, where the lookup shares each G2 slice among sixteen prefixes: with
// products of many multiplications, few rows for each and many prefixes at a time that decides.  Rows of
// 31,250 prefixes (4,096 prefixes) with n3 rows each, streamed / looked up, us:
//   rank 128, d = (4,4,8)   n3 = 1  1129 / 666 (151 / 152)    n3 = 16  1136 / 751 (157 / 153)
//                           n3 = 32 1162 / 1207 (176 / 209)
//   rank 128, d = (8,4,4)   n3 = 2  1350 / 884 (168 / 319)    n3 = 32  1706 / 1563 (216 / 268)
//   rank 128, d = (4,5,5)   n3 = 2  1340 / 1037 (176 / 243)   n3 = 8   1482 / 1498 (212 / 282)
//   ranks (300,40), d = (4,4,4)  n3 = 1  811 / 694 (94 / 153)
//   rank 64, d = (4,4,8)    n3 = 1  226 / 494 (35 / 123)
bool table_streamed(const Plan& pl, int64_t count) {
  const Shape& s = pl.sh;
  if (!pl.mfma && ((size_t)((kTableIds * s.S3 + 3) & ~3) + (size_t)s.M * (s.r2 + 1)) * 4 > kDirectLds)
    return false;
  const int64_t product = (int64_t)s.d1 * s.r1 * s.W;
  constexpr int64_t kTableProduct = 1 << 17, kTablePrefixes = 1 << 14;
  return product < kTableProduct || s.n3 > product >> (pl.mfma ? 14 : 16) ||
         std::min(count, pl.user_maxB) < kTablePrefixes * s.n3;
}

void launch_table(const Plan& pl, const float* g1, const float* g2, const float* g3, int64_t first,
                  int64_t count, float* out, hipStream_t st) {
  const Shape& s = pl.sh;
  const int n3 = (int)s.n3, p0 = (int)(first / n3), np = (int)((first + count - 1) / n3) - p0 + 1;
  // A launch of 2^32 threads or more is refused: a run of many prefixes takes several launches, each
  // long enough (a million blocks) for the gap between two not to count.
  constexpr int64_t kTableBlocks = 1 << 20;
  if (pl.mfma) {
    // enough wavefronts to fill the chip several times over, but no run so short that forming
    // the products (about R/8 tiles' worth of work) outweighs it
    const int upt = 16 / s.d3, tiles = cdiv(n3, upt), nvp = np * pl.split;
    const int per = s.r1 >= 128 ? 1 : s.r1 >= 64 ? 2 : 4;
    const int want = std::max(1, cdiv(8192, cdiv(nvp, per)));
    const int seg_tiles = std::min(tiles, std::max(cdiv(tiles, want), std::max(2, s.r1 / 8)));
    const int nseg = cdiv(tiles, seg_tiles);
    const int most = (int)std::min<int64_t>(nvp, kTableBlocks * kDWaves / nseg * per);
#define TT_TB(RR)                                                                                   \
  do {                                                                                              \
    if (s.d3 == 4)                                                                                  \
      k_table_mfma<RR, 4><<<grid, kDThreads, 0, st>>>((int)s.n2, n3, pl.split, (int)first, (int)count, \
                                                      vp, nv, nseg, seg_tiles, g1, g2, g3, out);    \
    else                                                                                            \
      k_table_mfma<RR, 8><<<grid, kDThreads, 0, st>>>((int)s.n2, n3, pl.split, (int)first, (int)count, \
                                                      vp, nv, nseg, seg_tiles, g1, g2, g3, out);    \
  } while (0)
    for (int64_t done = 0; done < nvp; done += most) {
      const int vp = (int)(p0 * pl.split + done), nv = (int)std::min<int64_t>(most, nvp - done);
      const int grid = cdiv((int64_t)cdiv(nv, per) * nseg, kDWaves);
      switch (s.r1) {
        case 8: TT_TB(8); break;
        case 16: TT_TB(16); break;
        case 32: TT_TB(32); break;
        case 64: TT_TB(64); break;
        default: TT_TB(128); break;
      }
    }
#undef TT_TB
    return;
  }
  const int want = std::max(1, cdiv(2048, np));
  const int seg_ids = cdiv(std::max(cdiv(n3, want), kTableIds), kTableIds) * kTableIds;
  const int nseg = cdiv(n3, seg_ids);
  const int most = (int)std::min<int64_t>(np, kTableBlocks / nseg);
  const size_t lds = ((size_t)((kTableIds * s.S3 + 3) & ~3) + (size_t)s.M * (s.r2 + 1)) * sizeof(float);
  for (int64_t done = 0; done < np; done += most)
    k_table_any<<<(int)std::min<int64_t>(most, np - done) * nseg, kDThreads, lds, st>>>(
        s, (int)first, (int)count, (int)(p0 + done), nseg, seg_ids, g1, g2, g3, out);
}

}  // namespace ttemb
