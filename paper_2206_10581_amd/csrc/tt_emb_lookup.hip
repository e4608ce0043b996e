// Lookups (no backward pass) of the matrix-core shapes with ranks up to 32 (gfx950, fp32): rows straight
// from the cores, with no prefix product in memory and no index structure behind the sort.
//
// The batch's ids come sorted by prefix, i2 in front of i1 (Plan::lookup_keys): neighbouring slots
// share a G2 slice, so a wavefront that takes a tile of slots forms the few products of its tile itself,
// from one G2 slice that it holds in registers.
#include <algorithm>

#include "tt_emb_internal.h"

namespace ttemb {

constexpr int kLThreads = 256;
constexpr int kLWaves = kLThreads / kWave;

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int value_at(int v, int src) {
  return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(src));
}
// lane `dst` of the result holds v (every lane names another destination)
__device__ __forceinline__ int push_to(int dst, int v) { return __builtin_amdgcn_ds_permute(dst * 4, v); }

// Trades between lanes l and l + 32: the lower lane ends with the x of both, the upper with the y of both.
__device__ __forceinline__ void swap_halves(float x, float y, float& of_lower, float& of_upper) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                  false, false);
  of_lower = __builtin_bit_cast(float, (uint32_t)r[0]);
  of_upper = __builtin_bit_cast(float, (uint32_t)r[1]);
}

// One wavefront per tile of TSL sorted slots.  Slabs (four lines of G1 each, `split` of them for
// d1 = 4*split) of the tile's distinct prefixes are taken up to four at a time, as many as share one i2:
//   P^T  (4R columns of G2[i2]) x (16 G1 lines): the G2 operand stays in registers while i2 does; the
//        columns of the output tiles are dealt so that a lane's four accumulators t = 0..3 are four
//        neighbours of a product's line: 16-byte loads of G2, 16-byte writes of P to LDS
//   E^T  (16/D3 ids x D3) x (16 lines of P): a lane's four accumulators are four neighbours of a row, so
//        rows go to memory from the registers, 16 bytes a lane, whole rows a store
// The terms of every sum are added in the order of the kernels with index structures (k_prefix_fwd_mfma
// adds k and R/2 + k side by side, k_row_fwd_mfma runs of R/4), so rows are bit-identical to theirs.
//
// Those kernels write and read a product per prefix (316 MB at 500,000 Zipf ids of n = (480,500,500),
// d = (8,4,4), rank 16) and need ids sorted in full, slab by slab, and prefixes grouped by i2: 62 + 134 us
// of arithmetic behind 166 us of index work, 366 us a lookup; here 90 behind 45.  Bound by the vector
// memory path where prefixes have one or two ids: lines of G1 and G3 loaded element by element took 134
// us instead of 113 with uniform ids.
template <int R, int D3, int TSL, bool AHEAD>
__global__ __launch_bounds__(kLThreads) void k_lookup_mfma(
    int B, int split, uint32_t n1, uint32_t sentinel, int i3_bits, const float* __restrict__ g1,
    const float* __restrict__ g2, const float* __restrict__ g3, const uint32_t* __restrict__ skey,
    const uint32_t* __restrict__ perm, float* __restrict__ out, Counters* ctr) {
  constexpr int W = 4 * R, S1 = 4 * R, S2 = R * W, S3 = R * D3, D = 16 * D3;
  constexpr int KQ = R / 4;             // contraction indices of a lane
  constexpr int NX = (W + 63) / 64;     // runs of 64 columns of P
  constexpr int UPT = 16 / D3;          // ids of a row product
  constexpr int RS = R + 4, PS = 16 * RS;  // LDS strides of a line and of a slab's product
  __shared__ __align__(16) float Pl[kLWaves][4 * PS];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int l16 = lane % 16, kg = lane / 16;
  float* P = Pl[w];
  const int tile = blockIdx.x * kLWaves + w;
  const int s = tile * TSL + lane;
  if (tile * TSL >= B) return;
  const bool in = lane < TSL && s < B;
  const uint32_t key = in ? skey[s] : sentinel;
  const uint32_t pos = in ? perm[s] : 0u;
  if (in && pos >= (uint32_t)B) atomicOr(&ctr->err, 4);
  const bool placed = in && pos < (uint32_t)B;
  // out-of-range ids (the tail of the sorted order) get zero rows
  unsigned long long zero_slots = __ballot(placed && key >= sentinel);
  while (zero_slots) {
    const int sl = __ffsll((long long)zero_slots) - 1;
    zero_slots &= zero_slots - 1;
    float* o = out + (size_t)(uint32_t)value_at((int)pos, sl) * split * D;
    for (int e = lane * 4; e < split * D; e += kWave * 4) *(f4*)(o + e) = f4{0.f, 0.f, 0.f, 0.f};
  }
  const int nv = __popcll(__ballot(in && key < sentinel));
  if (nv == 0) return;
  const uint32_t p = key >> i3_bits;
  const int i3 = lane < nv ? (int)(key & ((1u << i3_bits) - 1u)) : 0;
  const int i2 = (int)(p / n1), i1 = (int)(p - (uint32_t)i2 * n1);
  const uint32_t p_before = __shfl_up(p, 1);
  const unsigned long long starts = __ballot(lane < nv && (lane == 0 || p != p_before));
  const unsigned long long upto = starts & (lane == 63 ? ~0ull : ((2ull << lane) - 1ull));
  const int np = __popcll(starts), rank = __popcll(upto);  // rank: prefixes up to this lane's, itself included
  // lane e takes the tile's e-th prefix: its first slot, i1 and i2
  const bool first = (starts >> lane) & 1ull;
  const int dst = first ? rank - 1 : np + lane - rank;
  const int q_slot = push_to(dst, lane), q_i1 = push_to(dst, i1), q_i2 = push_to(dst, i2);
  // row products: every UPT-th slot of a prefix starts one
  const int run_first = 63 - __clzll((long long)(upto | 1ull));
  const unsigned long long groups = __ballot(lane < nv && (lane - run_first) % UPT == 0);

  // contraction order of the prefix products: k and R/2 + k side by side.  Lane group kg takes half kg%2
  // of a line of G1, its even (kg < 2) or odd elements
  const int k0 = (kg % 2) * (R / 2) + kg / 2;  // a lane's indices: k0, k0 + 2, ...
  const int wide = split < 4 ? split : 4;      // slabs of a prefix in a batch
  const int most = 4 / wide;                   // prefixes in a batch
  const int id = D3 == 4 ? kg : kg / 2;        // id of a row product that this lane stores
  // G1 lines of prefixes [pi, pi + nq), slabs from h0 on, as they lie in memory: line l16 is prefix pi +
  // l16/4/wide, slab h0 + l16/4%wide (absent ones repeat one that is there); lanes kg and kg + 2 load a quarter
  // line each (rank 8 element by element)
  constexpr int NV = KQ % 4 == 0 ? KQ / 4 : 1;
  const int my_q = l16 / 4 / wide, my_h = l16 / 4 - my_q * wide;
  f4 av[NV];
  auto load_lines = [&](int pi, int nq, int h0) {
    const int qi = min(pi + my_q, pi + nq - 1), h = min(h0 + my_h, split - 1);
    const float* line = g1 + ((size_t)__shfl(q_i1, qi) * split + h) * S1 + (l16 % 4) * R;
    if constexpr (KQ % 4 == 0) {
#pragma unroll
      for (int j = 0; j < KQ / 4; ++j) av[j] = ((const f4*)(line + (kg % 2) * (R / 2) + (kg / 2) * KQ))[j];
    } else {
#pragma unroll
      for (int j = 0; j < KQ; ++j) av[0][j] = line[k0 + 2 * j];
    }
  };
  // slices of G3 of the row product whose first slot is `at`, as they lie in memory: a quad loads a 4 x 4 block by
  // lines
  f4 cv[NV];
  auto end_of = [&](int at) {  // the next product's first slot or the next prefix's
    const unsigned long long after = groups & ~((2ull << at) - 1ull);
    return after ? __ffsll((long long)after) - 1 : nv;
  };
  const int j3 = l16 % D3;
  auto load_slices = [&](int at) {
    const int slot = min(at + l16 / D3, end_of(at) - 1);
    const float* C = g3 + (size_t)__shfl(i3, slot) * S3 + (KQ * kg) * D3;
    if constexpr (KQ % 4 == 0) {
#pragma unroll
      for (int j = 0; j < KQ / 4; ++j) cv[j] = *(const f4*)(C + (4 * j + j3 % 4) * D3 + j3 / 4 * 4);
    } else {
#pragma unroll
      for (int j = 0; j < KQ; ++j) cv[0][j] = C[j * D3 + j3];
    }
  };
  auto prefixes_from = [&](int pi) {
    int nq = 1;
    if (pi < np) {
      const int bin = value_at(q_i2, pi);
      while (nq < most && pi + nq < np && value_at(q_i2, pi + nq) == bin) ++nq;
    }
    return nq;
  };

  f4 b2[NX][KQ];
  int have = -1;  // i2 of b2
  int nq = prefixes_from(0);
  if constexpr (AHEAD) {
    load_lines(0, nq, 0);
    load_slices(0);
  }
  for (int pi = 0; pi < np;) {
    const int bin = value_at(q_i2, pi);
    if (bin != have) {
      have = bin;
      const float* Bm = g2 + (size_t)bin * S2;
#pragma unroll
      for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int j = 0; j < KQ; ++j)
          b2[x][j] = *(const f4*)(Bm + (size_t)(k0 + 2 * j) * W + x * 64 + 4 * (W < 64 ? l16 % (W / 4) : l16));
    }
    // slots of the batch
    const int f0 = value_at(q_slot, pi), f1 = pi + nq < np ? value_at(q_slot, pi + nq) : nv;
    const unsigned long long here = groups & (f1 >= 64 ? ~0ull : (1ull << f1) - 1ull) & ~((1ull << f0) - 1ull);
    const int next_nq = prefixes_from(pi + nq);
    for (int h0 = 0; h0 < split; h0 += wide) {  // one round up to d1 = 16
      {
        if constexpr (!AHEAD) load_lines(pi, nq, h0);
        float a[KQ];
        if constexpr (KQ % 4 == 0) {
          // lanes kg and kg + 2 trade the odd elements of one for the even ones of the other
#pragma unroll
          for (int j = 0; j < KQ / 4; ++j) {
            swap_halves(av[j].x, av[j].y, a[2 * j], a[KQ / 2 + 2 * j]);
            swap_halves(av[j].z, av[j].w, a[2 * j + 1], a[KQ / 2 + 2 * j + 1]);
          }
        } else {
#pragma unroll
          for (int j = 0; j < KQ; ++j) a[j] = av[0][j];
        }
        if constexpr (AHEAD) {  // the next lines are in flight while these are used
          if (h0 + wide < split) load_lines(pi, nq, h0 + wide);
          else if (pi + nq < np) load_lines(pi + nq, next_nq, 0);
        }
        f4 acc[NX][4];
#pragma unroll
        for (int x = 0; x < NX; ++x)
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[x][t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KQ; ++j)
#pragma unroll
          for (int x = 0; x < NX; ++x)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[x][t] = mfma4(b2[x][j][t], a[j], acc[x][t]);
        // acc[x][t][v]: column 64x + 16kg + 4v + t of line l16
        wave_sync();  // the previous batch's products have been read
#pragma unroll
        for (int x = 0; x < NX; ++x)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int col = 64 * x + 16 * kg + 4 * v;
            if (W >= 64 || col < W)
              *(f4*)(P + (l16 / 4) * PS + ((l16 % 4) * 4 + col / R) * RS + col % R) =
                  f4{acc[x][0][v], acc[x][1][v], acc[x][2][v], acc[x][3][v]};
          }
        wave_sync();
      }
      for (unsigned long long todo = here; todo; todo &= todo - 1) {
        const int at = __ffsll((long long)todo) - 1, end = end_of(at), n = end - at;
        const int qi = value_at(rank, at) - 1 - pi;
        if constexpr (!AHEAD) load_slices(at);
        float c[KQ];  // c[j] = G3[KQ*kg + j][j3]
        if constexpr (KQ % 4 == 0) {
#pragma unroll
          for (int j = 0; j < KQ / 4; ++j) {
            const f4 t = quad_turned(cv[j], lane);
            c[4 * j] = t.x;
            c[4 * j + 1] = t.y;
            c[4 * j + 2] = t.z;
            c[4 * j + 3] = t.w;
          }
        } else {
#pragma unroll
          for (int j = 0; j < KQ; ++j) c[j] = cv[0][j];
        }
        if constexpr (AHEAD) {
          // products follow each other in slot order; a further round of slabs begins with this batch's first
          if ((todo & (todo - 1)) == 0 && h0 + wide < split) load_slices(f0);
          else if (end < nv) load_slices(end);
        }
        const uint32_t row = (uint32_t)__shfl((int)pos, min(at + id, 63));
        const bool on = id < n && row < (uint32_t)B;
        for (int y = 0; y < wide && h0 + y < split; ++y) {
          const float* pr = P + (qi * wide + y) * PS + l16 * RS + KQ * kg;
          float b[KQ];
          if constexpr (KQ % 4 == 0) {
#pragma unroll
            for (int j = 0; j < KQ / 4; ++j) {
              const f4 v = ((const f4*)pr)[j];
              b[4 * j] = v.x;
              b[4 * j + 1] = v.y;
              b[4 * j + 2] = v.z;
              b[4 * j + 3] = v.w;
            }
          } else {
#pragma unroll
            for (int j = 0; j < KQ; ++j) b[j] = pr[j];
          }
          f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < KQ; ++j) acc = mfma4(c[j], b[j], acc);
          // acc[v]: entry 4kg + v of the 16 (id, j3), line l16 of the slab
          if (on)
            __builtin_nontemporal_store(
                acc, (f4*)(out + ((size_t)row * split + h0 + y) * D + l16 * D3 + (D3 == 8 ? 4 * (kg % 2) : 0)));
        }
      }
    }
    pi += nq;
    nq = next_nq;
  }
}

// Counters of a lookup from its keys, sorted by prefix only, for tt_emb_get_stats; the keys are only read.
// A wavefront counts the prefixes that begin in its run of slots, 64 slots at a time.  Whether an id was met
// before: inside the 64 by comparing keys, in a prefix that goes on from slots before them by one bit of LDS
// for each i3.
constexpr int kCountSteps = 8;

__global__ __launch_bounds__(kLThreads) void k_count_lookup(const uint32_t* __restrict__ skey, int B,
                                                            uint32_t sentinel, int i3_bits,
                                                            Counters* __restrict__ ctr) {
  __shared__ uint32_t met[kLWaves][kMaxBins / 32];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int begin = (blockIdx.x * kLWaves + w) * kCountSteps * kWave, end = min(begin + kCountSteps * kWave, B);
  if (begin >= B) return;
  uint32_t* bits = met[w];
  uint32_t u = 0, q = 0, valid = 0;
  bool open = false, more = true;  // a prefix of this wavefront goes on; something is left to count
  uint32_t last = begin > 0 ? skey[begin - 1] : sentinel;  // key in front of the 64 (the first of all: none)
  for (int at0 = begin; more; at0 += kCountSteps * kWave) {
    uint32_t keys[kCountSteps];
#pragma unroll
    for (int j = 0; j < kCountSteps; ++j) keys[j] = skey[min(at0 + j * kWave + lane, B - 1)];
    for (int j = 0; j < kCountSteps && more; ++j) {
      const int at = at0 + j * kWave;
      uint32_t key = keys[0];
#pragma unroll
      for (int k = 1; k < kCountSteps; ++k) key = j == k ? keys[k] : key;
      const bool on = at + lane < B && key < sentinel;  // in-range ids lie in front
      uint32_t before = __shfl_up(key, 1);
      if (lane == 0) before = last;
      last = (uint32_t)value_at((int)key, 63);
      const unsigned long long starts = __ballot(on && (at + lane == 0 || key >> i3_bits != before >> i3_bits));
      const int nv = __popcll(__ballot(on)), first = starts ? __ffsll((long long)starts) - 1 : nv;
      const uint32_t i3 = key & ((1u << i3_bits) - 1u), word = i3 / 32 % (kMaxBins / 32), bit = 1u << i3 % 32;
      if (open && lane < first) u += !(atomicOr(&bits[word], bit) & bit);
      if (at < end) {
        bool seen = false;
        for (int k = 0; k < 63; ++k) seen |= k < lane && (uint32_t)value_at((int)key, k) == key;
        u += on && lane >= first && !seen;
        q += (starts >> lane) & 1ull;
        valid += on;
        if (starts) {  // the last prefix may go on
          wave_sync();
          for (int k = lane; k < kMaxBins / 32; k += kWave) bits[k] = 0u;
          wave_sync();
          if (on && lane >= 63 - __clzll((long long)starts)) atomicOr(&bits[word], bit);
          open = true;
        }
      }
      more = nv == kWave && (at + kWave < end || (open && !(at >= end && starts)));
    }
  }
  u = wave_inclusive_scan(u, lane);
  q = wave_inclusive_scan(q, lane);
  valid = wave_inclusive_scan(valid, lane);
  if (lane == 63) {
    atomicAdd((uint32_t*)&ctr->U, u);
    atomicAdd((uint32_t*)&ctr->Q, q);
    atomicAdd((uint32_t*)&ctr->nvalid, valid);
  }
}

__global__ void k_clear_counts(Counters* ctr) { ctr->U = ctr->Q = ctr->nvalid = 0; }

bool lookup_shape(const Shape& s) { return s.r1 <= 32; }

// Slots of a wavefront's tile.  Short tiles put more wavefronts in flight and shorten the chain of batches
// of each; long ones load a G2 slice (16 KiB at rank 32) for more rows.  Kernel times in us with 16 / 32 /
// 64 slots, uniform ids: rank 16, n = (480,500,500), d = (8,4,4): 50,000 ids 35 / 41 / 58, 200,000 76 / 80 /
// 96, 500,000 118 / 114 / 121; rank 32, n = 136^3, d = (4,4,8): 9,000 ids 46 / 59 / 85, 50,000 32 / 31 / 38,
// 200,000 63 / 56 / 60, 500,000 140 / 111 / 96.
static int lookup_tile(const Shape& s, int B) {
  if (s.r1 <= 16) return B <= kSmallBatch ? 16 : 32;
  return B <= kSmallBatch / 16 ? 16 : B <= kSmallBatch ? 32 : 64;
}
// The next batch's lines of G1 and the next product's slices of G3 are loaded ahead where tiles are short at rank
// 32: few wavefronts a compute unit, whose chain of loads is the time.  Elsewhere other wavefronts fill the waits,
// and what keeping loads in flight takes in instructions and registers is lost.  Lookups in us without / with,
// uniform ids: rank 32, 8,500 ids of (480,500,500) x (8,4,4) 48.3 / 48.0, Zipf 49.1 / 48.4, of 60^3 x (16,4,4)
// 52.9 / 51.9, of 136^3 38.9 / 39.0; longer tiles, 30,000 ids of 136^3 46.3 / 47.1, 90,000 52.2 / 63.1, of
// (480,500,500) x (8,4,4) 121 / 153; rank 16, 90,000 of 136^3 38.4 / 41.2, rank 8 35.7 / 37.0.
void launch_lookup(const Plan& pl, const Workspace& ws, const float* g1, const float* g2, const float* g3, int B,
                   float* out, hipStream_t st) {
  const int f = pl.lookup_keys.sorted();
  auto launch = [&](auto kernel, int slots) {
    kernel<<<(B + kLWaves * slots - 1) / (kLWaves * slots), kLThreads, 0, st>>>(
        B, pl.split, pl.user_n1, pl.lookup_keys.sentinel, pl.lookup_i3_bits, g1, g2, g3, ws.key[f], ws.val[f],
        out, ws.ctr);
  };
  const int tile = lookup_tile(pl.sh, B);
  auto by_d3 = [&](auto k4, auto k8, int slots) { pl.sh.d3 == 4 ? launch(k4, slots) : launch(k8, slots); };
  // the grid is made for the slots of the kernel that is launched
#define TT_TILE(R_, T_, A_) by_d3(k_lookup_mfma<R_, 4, T_, A_>, k_lookup_mfma<R_, 8, T_, A_>, T_)
#define TT_RANK(R_) if (tile == 16) TT_TILE(R_, 16, false); else TT_TILE(R_, 32, false)
  switch (pl.sh.r1) {
    case 8: TT_RANK(8); break;
    case 16: TT_RANK(16); break;
    default:
      if (tile == 16) TT_TILE(32, 16, true);
      else if (tile == 32) TT_TILE(32, 32, false);
      else TT_TILE(32, 64, false);
  }
#undef TT_RANK
#undef TT_TILE
}

void launch_count_lookup(const Plan& pl, const Workspace& ws, int B, hipStream_t st) {
  constexpr int kSlots = kLWaves * kCountSteps * kWave;
  k_clear_counts<<<1, 1, 0, st>>>(ws.ctr);
  k_count_lookup<<<(B + kSlots - 1) / kSlots, kLThreads, 0, st>>>(ws.key[pl.lookup_keys.sorted()], B,
                                                                 pl.lookup_keys.sentinel, pl.lookup_i3_bits, ws.ctr);
}

}  // namespace ttemb
