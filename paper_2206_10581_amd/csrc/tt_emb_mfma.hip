// Matrix-core (MFMA) kernels for the table shapes d1 = d2 = 4, r1 = r2 = R in {8, 16, 32, 64, 128},
// d3 in {4, 8}: the partial product of a row is then 16 x R, and once ids that share an (i1,i2)
// prefix, an i2 or an i3 are stacked (paper Section 4.2: they share core slices) every step of the
// path is a dense contraction with a 16- or 32-wide side.
//
// Lane layouts used below (wave64):
//   v_mfma_f32_32x32x2f32   A[i][k]: i = lane%32, k = lane/32     B[k][j]: k = lane/32, j = lane%32
//                           D[i][j]: i = 8*(v/4) + 4*(lane/32) + v%4, j = lane%32, v = 0..15
//   v_mfma_f32_16x16x4f32   A[i][k]: i = lane%16, k = lane/16     B[k][j]: k = lane/16, j = lane%16
//                           D[i][j]: i = 4*(lane/16) + v, j = lane%16, v = 0..3
// The summation index k may be enumerated in any order as long as A and B agree, so each lane
// takes a contiguous run of k (vector loads) instead of the strided one the raw layout suggests.
#include <algorithm>
#include <type_traits>

#include "tt_emb_internal.h"

namespace ttemb {

typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int kMThreads = 256;
constexpr int kMWaves = kMThreads / kWave;

__device__ __forceinline__ f16v mfma32(float a, float b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma16(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ const float* grad_row_ptr(int code, const float* __restrict__ grad,
                                                     const float* __restrict__ gsum, int D) {
  // code >= 0: batch position of the id's only occurrence; else row -(code+1) of the per-id sums
  return code >= 0 ? grad + (size_t)code * D : gsum + (size_t)(-code - 1) * D;
}

typedef float f2 __attribute__((ext_vector_type(2)));

// Value of v in lane `src`, where src is the same for the whole wavefront (a scalar read, no LDS).
__device__ __forceinline__ int lane_value(int v, int src) {
  return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(src));
}

// A value that is the same in all lanes, as a scalar.
__device__ __forceinline__ int wave_value(int v) { return __builtin_amdgcn_readfirstlane(v); }

// One lane's share (VPL consecutive floats, VPL = 1 or 2) of a row, moved with a single non-temporal
// access: rows of grad_out are streamed once and should not displace the intermediates that the path does
// re-read.
template <int VPL>
__device__ __forceinline__ void stream_load(const float* src, float* v) {
  if constexpr (VPL == 2) {
    const f2 t = __builtin_nontemporal_load((const f2*)src);
    v[0] = t.x;
    v[1] = t.y;
  } else {
    v[0] = __builtin_nontemporal_load(src);
  }
}

#define TT_ZERO16 {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}

// All kernels below are written as "issue every load of a work item, then compute": the loads of a
// phase sit in one straight-line block that ends in sched_barrier(0), so the compiler cannot sink
// them next to their uses (which would serialise their latencies); out-of-range lanes read a
// clamped, valid address and their values are discarded by a select.
#define TT_LOADS_DONE() __builtin_amdgcn_sched_barrier(0)

// ---------------------------------------------------------------------------------------------
// P_q = G1[i1] G2[i2] for the <= 16 prefixes of one by-i2 chunk: rows of up to eight G1 slices
// stacked (32 x R) times the chunk's G2 slice (R x 4R).  A work unit is (chunk, a share of the 4R
// output columns); one single-wavefront block per unit, so that the units spread evenly over all
// SIMDs.
// Units per chunk: two or four side by side over the 32-column tiles of the product (four shorten
// the kernel at rank 32 by a fifth; splitting the sixteen prefixes of a chunk over units as well
// only re-reads the G2 slice, which costs more than it gains).  Ranks 64 and 128 take
// k_prefix_fwd_wide.
constexpr int pf_units(int R) { return R >= 32 ? 4 : 2; }

template <int R>
__global__ __launch_bounds__(kWave) void k_prefix_fwd_mfma(
    const float* __restrict__ g1, const float* __restrict__ g2, const int4* __restrict__ c2_item,
    const int4* __restrict__ c2_desc, float* __restrict__ P, const Counters* __restrict__ ctr) {
  constexpr int W = 4 * R, PN = 16 * R, S1 = 4 * R, S2 = R * W, KH = R / 2, NT = W / 32;
  constexpr int kPfUnits = pf_units(R);
  constexpr int UC = kPfUnits < NT ? kPfUnits : NT;  // units side by side over the columns
  constexpr int UM = kPfUnits / UC;                  // 1: both row tiles in one unit, 2: one each
  constexpr int NTH = NT / UC, MTH = 2 / UM;         // column and row tiles of one unit
  const int lane = threadIdx.x, half = lane / 32, l32 = lane % 32;
  // one block per possible unit: the grid never exceeds the tables
  const int nchunk = ctr->nchunk2, unit = blockIdx.x;
  const int c = unit / kPfUnits, sub = unit % kPfUnits;
  const int nt0 = (sub / UM) * NTH, mt0 = (sub % UM) * MTH;
  // the chunk's records and descriptor are read together with the count
  const int4 item = c2_item[(size_t)c * kChunk2 + lane % kChunk2];
  const int4 desc = c2_desc[c];
  if (c >= nchunk) return;
  const int bin = desc.x, cnt = desc.z;
  if (mt0 * 8 >= cnt) return;  // the chunk has no prefix in this unit's row tile
  const float* Bm = g2 + (size_t)bin * S2 + (size_t)(KH * half) * W + nt0 * 32 + l32;
  float b[NTH][KH];
#pragma unroll
  for (int t = 0; t < NTH; ++t)
#pragma unroll
    for (int j = 0; j < KH; ++j) b[t][j] = Bm[(size_t)j * W + t * 32];
  const bool mine = lane < cnt;  // records past the chunk's count are unwritten
  const int myq = mine ? item.x : -1;
  const int myi1 = mine ? item.y : 0;
  float a[MTH][KH];
#pragma unroll
  for (int mt = 0; mt < MTH; ++mt) {
    const int ql = (mt0 + mt) * 8 + l32 / 4, j1 = l32 % 4;
    const int q = __shfl(myq, ql), i1 = __shfl(myi1, ql);
    const f4* src = (const f4*)(g1 + (size_t)i1 * S1 + j1 * R + KH * half);
#pragma unroll
    for (int j = 0; j < KH / 4; ++j) {
      f4 v = src[j];
      a[mt][4 * j + 0] = q >= 0 ? v.x : 0.f;
      a[mt][4 * j + 1] = q >= 0 ? v.y : 0.f;
      a[mt][4 * j + 2] = q >= 0 ? v.z : 0.f;
      a[mt][4 * j + 3] = q >= 0 ? v.w : 0.f;
    }
  }
  int qrow[MTH][4];  // prefix of accumulator rows v/4 of each row tile
#pragma unroll
  for (int mt = 0; mt < MTH; ++mt)
#pragma unroll
    for (int x = 0; x < 4; ++x) qrow[mt][x] = __shfl(myq, (mt0 + mt) * 8 + 2 * x + half);
  TT_LOADS_DONE();
#pragma unroll
  for (int t = 0; t < NTH; ++t) {
#pragma unroll
    for (int mt = 0; mt < MTH; ++mt) {
      if ((mt0 + mt) * 8 >= cnt) break;
      f16v acc = TT_ZERO16;
#pragma unroll
      for (int j = 0; j < KH; ++j) acc = mfma32(a[mt][j], b[t][j], acc);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int q = qrow[mt][v / 4];
        if (q >= 0) P[(size_t)q * PN + (v % 4) * W + (nt0 + t) * 32 + l32] = acc[v];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Ranks 64 and 128: a G2 slice has 64 to 256 KiB, and the products of the prefixes are large enough for
// the rate of the matrix cores to count.  An fp32 number is the sum of three bf16 numbers (8 + 8 + 8
// significant bits, each rounded to nearest), and bf16 products run sixteen times as fast as fp32 ones, so
// a product of two such sums is formed as its six largest terms: hi*hi, hi*mid, mid*hi, mid*mid, hi*lo,
// lo*hi, each exact and added up in fp32.  What is left out is at most 2^-24.2 of a term (rms 2^-27.5), of
// either sign;
// the error against 64 bits is that of the fp32 instructions or less (relative 2-norms, fp32 -> this: rank
// 128, 20,000 uniform ids of (60,50,40) x (8,4,4), rows 2.87e-7 -> 2.61e-7, G1 4.30e-7 -> 4.16e-7, G2 1.83e-7 ->
// 1.59e-7, G3 3.26e-7 -> 2.98e-7; with all numbers of one sign 1.72e-7 -> 1.72e-7 and 6.8e-8 -> 6.2e-8 for G2).
//
// Splits do not hold for infinities, for numbers that round up to one, and for numbers so small that their
// lower parts leave the range of bf16 (below 2^-102 and not zero).  The first two leave NaN or an infinity in the
// result, and so that products stay in range it is looked at for very small numbers as well (recheck); the last
// are found before they are split (some_inexact).  A wavefront that finds either forms its tile anew with fp32
// instructions.  The gradient kernel is bound by the vector ALUs and looks for small operands only if the forward
// has met one in the cores or u_bwd_role in dPsum (Counters::small); looking always cost it 7 %.
typedef __bf16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 h4 __attribute__((ext_vector_type(4)));
typedef __bf16 h8 __attribute__((ext_vector_type(8)));
template <class V>
struct Split {
  V hi, mid, lo;
};
__device__ __forceinline__ void split_two(float x, float y, h2& hi, h2& mid, h2& lo) {
  const f2 v = {x, y};
  hi = __builtin_convertvector(v, h2);
  const f2 r = v - __builtin_convertvector(hi, f2);  // exact, as is the next one
  mid = __builtin_convertvector(r, h2);
  lo = __builtin_convertvector(r - __builtin_convertvector(mid, f2), h2);
}
__device__ __forceinline__ Split<h4> split_four(f4 v) {
  h2 a[3], b[3];
  split_two(v.x, v.y, a[0], a[1], a[2]);
  split_two(v.z, v.w, b[0], b[1], b[2]);
  return {__builtin_shufflevector(a[0], b[0], 0, 1, 2, 3), __builtin_shufflevector(a[1], b[1], 0, 1, 2, 3),
          __builtin_shufflevector(a[2], b[2], 0, 1, 2, 3)};
}
__device__ __forceinline__ Split<h8> split_eight(const float* v) {
  const Split<h4> a = split_four(f4{v[0], v[1], v[2], v[3]}), b = split_four(f4{v[4], v[5], v[6], v[7]});
  return {__builtin_shufflevector(a.hi, b.hi, 0, 1, 2, 3, 4, 5, 6, 7),
          __builtin_shufflevector(a.mid, b.mid, 0, 1, 2, 3, 4, 5, 6, 7),
          __builtin_shufflevector(a.lo, b.lo, 0, 1, 2, 3, 4, 5, 6, 7)};
}
// acc += A B, 32 x 16 times 16 x 32: half a wavefront holds eight k each, A[i][k]: i = lane%32, B[k][j]:
// j = lane%32, D as of v_mfma_f32_32x32x2f32
__device__ __forceinline__ f16v mfma_split(const Split<h8>& a, const Split<h8>& b, f16v acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo, b.hi, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, b.lo, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.mid, b.mid, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.mid, b.hi, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, b.mid, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, b.hi, acc, 0, 0, 0);
}
// Whether one of N operands is below 2^-102 and not zero.  Half an instruction each (the smallest magnitude of all
// in pairs) unless one is that small or zero.
constexpr float kExactFrom = 0x1p-102f;
template <int N>
__device__ __forceinline__ bool some_inexact(const float* v) {
  static_assert(N % 2 == 0, "in pairs");
  float least = kExactFrom;
#pragma unroll
  for (int i = 0; i < N; i += 2) asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(least) : "v"(v[i]), "v"(v[i + 1]));
  bool found = false;
  if (least < kExactFrom) {
#pragma unroll
    for (int i = 0; i < N; ++i) found |= v[i] != 0.f && fabsf(v[i]) < kExactFrom;
  }
  return found;
}
// Whether some entry is not finite, or below 2^-80 and not zero.
__device__ __forceinline__ bool recheck(const f16v& acc) {
  uint32_t most = 0u, least = ~0u;  // of the magnitudes, of those that are not zero less one
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const float f = acc[v];  // (a vector's element is not cast in place: the compiler casts its first one)
    const uint32_t x = __builtin_bit_cast(uint32_t, f) & 0x7fffffffu;
    most = max(most, x);
    least = min(least, x - 1u);
  }
  return __ballot(most >= 0x7f800000u || least + 1u < (127u - 80u) << 23 && least != ~0u) != 0ull;
}
// Eight bf16 of a line in LDS, of each of the three planes
template <int PLANE>
__device__ __forceinline__ Split<h8> split_from(const __bf16* at) {
  return {*(const h8*)at, *(const h8*)(at + PLANE), *(const h8*)(at + 2 * PLANE)};
}

// P_q for the <= 16 prefixes of a by-i2 chunk.  A block of four wavefronts takes a chunk's 64 lines times
// 128 columns: the lines are split and staged in LDS once for all four, every wavefront takes a strip of 32
// columns of G2 straight to registers, splits it and uses it for both tiles of 32 lines.  At most as many
// blocks as the device holds walk the units: the grid is sized for the most chunks a batch could have, and
// dispatching blocks that find nothing cost more than the work.
template <int R>
__global__ __launch_bounds__(kMThreads, 3) void k_prefix_fwd_wide(
    const float* __restrict__ g1, const float* __restrict__ g2, const int4* __restrict__ c2_item,
    const int4* __restrict__ c2_desc, float* __restrict__ P, Counters* __restrict__ ctr) {
  static_assert(R == 64 || R == 128, "columns of a block divide the product");
  constexpr int W = 4 * R, PN = 16 * R, S1 = 4 * R, S2 = R * W, KT = R / 16;
  constexpr int UN = W / 128;  // blocks side by side over the columns
  constexpr int AS = R + 8, PL = 64 * AS;  // stride of a line and of a plane in LDS
  __shared__ __align__(16) __bf16 As[3 * PL];
  __shared__ int q_of[kChunk2], i1_of[kChunk2], inexact;
  const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave, half = lane / 32, l32 = lane % 32;
  const int nunit = ctr->nchunk2 * UN;
  for (int unit = blockIdx.x; unit < nunit; unit += gridDim.x) {
    const int c = unit / UN, col = (unit % UN) * 128 + w * 32 + l32;
    const int4 desc = c2_desc[c];
    const int cnt = desc.z;
    __syncthreads();  // the previous unit's readers of As are done
    if (tid < kChunk2) {
      // records past the chunk's count are unwritten
      const int4 item = c2_item[(size_t)c * kChunk2 + min(tid, cnt - 1)];
      q_of[tid] = item.x;
      i1_of[tid] = item.y;
    }
    if (tid == 0) inexact = 0;
    const float* Bm = g2 + (size_t)desc.x * S2 + col;
    float b[KT][8];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int j = 0; j < 8; ++j) b[t][j] = Bm[(size_t)(16 * t + 8 * half + j) * W];
    __syncthreads();
    // lines of prefixes past the count repeat the last one; they are not stored
    f4 row[R / 16];
#pragma unroll
    for (int i = 0; i < R / 16; ++i) {
      const int e = tid + i * kMThreads;  // 16-byte word of the 64 lines
      row[i] = ((const f4*)(g1 + (size_t)wave_value(i1_of[e / R]) * S1))[e % R];
    }
    TT_LOADS_DONE();
    if (some_inexact<R / 4>((const float*)row)) inexact = 1;
#pragma unroll
    for (int i = 0; i < R / 16; ++i) {
      const int e = (tid + i * kMThreads) * 4;
      const Split<h4> x = split_four(row[i]);
      __bf16* to = As + (e / R) * AS + e % R;
      *(h4*)to = x.hi;
      *(h4*)(to + PL) = x.mid;
      *(h4*)(to + 2 * PL) = x.lo;
    }
    const bool small_cols = __ballot(some_inexact<KT * 8>(&b[0][0])) != 0ull;
    __syncthreads();
    if ((small_cols || inexact) && lane == 0) atomicOr(&ctr->small, 1);
    f16v acc[2] = {TT_ZERO16, TT_ZERO16};
    const bool two = cnt > 8;  // uniform: the second tile has a prefix
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const Split<h8> y = split_eight(b[t]);
      const __bf16* at = As + l32 * AS + 16 * t + 8 * half;
      acc[0] = mfma_split(split_from<PL>(at), y, acc[0]);
      if (two) acc[1] = mfma_split(split_from<PL>(at + 32 * AS), y, acc[1]);
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      if (mt * 8 >= cnt) break;
      if (recheck(acc[mt]) || small_cols || inexact) {
        const float* ar = g1 + (size_t)i1_of[mt * 8 + l32 / 4] * S1 + (l32 % 4) * R + half * (R / 2);
        const float* br = Bm + (size_t)(half * (R / 2)) * W;
        acc[mt] = TT_ZERO16;
#pragma unroll 4
        for (int j = 0; j < R / 2; ++j) acc[mt] = mfma32(ar[j], br[(size_t)j * W], acc[mt]);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int ql = mt * 8 + 2 * (v / 4) + half;
        if (ql < cnt) P[(size_t)q_of[ql] * PN + (v % 4) * W + col] = acc[mt][v];
      }
    }
  }
}

// Gradients at prefix level.  Units of work, one block of four wavefronts each, walked with the grid's
// stride:
//   dG2   a group of chunks (wide_group) of one i2 and 128 columns: sum over the prefixes q of
//         G1[i1(q)]^T dPsum_q, R x 128.  The G1 lines of a chunk are split and staged in LDS, transposed,
//         for all four wavefronts, dPsum goes straight to registers (each value is used for R/32 tiles),
//         and the sum stays in registers from chunk to chunk: a chunk's 64 terms are one chain, the
//         chunks another (all in one chain, the error of dG2 was 2.1 times as large at 200,000 uniform
//         ids of rank 64).
//   dG1   a chunk: dg1part[q] = dPsum_q Bm^T, 64 x R with 4R to contract, 32 at a time through LDS.
// The units of a group follow each other, dG2 first: dPsum is then read again while it is near (rank 64,
// 500,000 uniform ids: all dG2 units first 530 us, so 510).  Measured with fp32 instructions before / bf16
// parts now: rank 128, 500,000 ids of (480,500,500) x (8,4,4), uniform 4440 / 3420 us, Zipf 970 / 700; rank
// 64, (480,480,482) x (4,4,8), uniform 563 / 456, Zipf 145 / 121.  The matrix cores are busy a third of the
// time; neither loads a chunk ahead nor two chunks side by side changed it: what remains is dPsum, read
// twice in pieces of 128 bytes to 2 KiB.
template <int R>
__global__ __launch_bounds__(kMThreads, 2) void k_prefix_bwd_wide(
    const float* __restrict__ g1, const float* __restrict__ g2, const float* __restrict__ dPsum,
    const int4* __restrict__ c2_item, const int4* __restrict__ c2_desc, float* __restrict__ dg1part,
    float* __restrict__ part2, const Counters* __restrict__ ctr) {
  static_assert(R == 64 || R == 128, "columns of a block divide the slice");
  constexpr int W = 4 * R, PN = 16 * R, S1 = 4 * R, S2 = R * W, UN = W / 128;
  constexpr int KD = 32, KS = KD + 8;  // depth of a step of the dG1 product, stride of its lines in LDS
  constexpr int TS = 64 + 8;           // stride of a column of G1 in LDS
  constexpr int PL2 = R * TS, PL1 = (64 + R) * KS, kLds = 3 * (PL2 > PL1 ? PL2 : PL1);
  __shared__ __align__(16) __bf16 L[kLds];
  __shared__ int q_of[kChunk2], i1_of[kChunk2], inexact;
  const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave, half = lane / 32, l32 = lane % 32;
  const int nchunk = ctr->nchunk2, grp = wide_group(nchunk, R);
  const int per_group = UN + grp, nunit = (nchunk + grp - 1) / grp * per_group;
  // records of chunk c; those past its count are unwritten and repeat the last one
  auto chunk_records = [&](int c, int cnt) {
    __syncthreads();  // the readers of the previous chunk's records and LDS tiles are done
    if (tid < kChunk2) {
      const int4 item = c2_item[(size_t)c * kChunk2 + min(tid, cnt - 1)];
      q_of[tid] = item.x;
      i1_of[tid] = item.y;
    }
    if (tid == 0) inexact = 0;
    __syncthreads();
  };
  // look for small operands or not: one form with a test at every product took 4 % longer (500,000 Zipf ids of
  // (480,500,500) x (8,4,4), rank 128; without any test 2376 us, one form 2410, two 2315)
  auto walk = [&](auto look) {
    for (int unit = blockIdx.x; unit < nunit; unit += gridDim.x) {
      const int c0 = unit / per_group * grp, c1 = min(c0 + grp, nchunk), sub = unit % per_group;
      if (sub < UN) {
        constexpr int MT = R / 32;
        const int col = sub * 128 + w * 32 + l32;
        f16v sum[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) sum[mt] = TT_ZERO16;
        int first = c0;  // where the running sum began
        int4 desc = c2_desc[c0];
        for (int c = c0; c < c1; ++c) {
          const int cnt = desc.z, bin = desc.x;
          chunk_records(c, cnt);
          // a step contracts four prefixes; half h takes lines 2h and 2h + 1 of each, so that addresses are a
          // scalar and a lane's offset.  Prefixes past the count count zero (their G1 lines are cleared) and
          // read the last one's dPsum.
          float b[4][8];
          const uint32_t bo = 2 * half * W + col;
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j)
              b[t][j] = (dPsum + (size_t)wave_value(q_of[4 * t + j / 2]) * PN + j % 2 * W)[bo];
          const int4 next = c2_desc[min(c + 1, nchunk - 1)];
          // eight lines of a column a thread, R/32 times: those of half k8 % 2 in step k8 / 2
          float a[R / 32][8];
          const uint32_t ao = tid % R;
#pragma unroll
          for (int i = 0; i < R / 32; ++i) {
            const int k8 = wave_value((tid + i * kMThreads) / R);
#pragma unroll
            for (int j = 0; j < 8; ++j)
              a[i][j] = (g1 + (size_t)wave_value(i1_of[k8 / 2 * 4 + j / 2]) * S1 + (k8 % 2 * 2 + j % 2) * R)[ao];
          }
          TT_LOADS_DONE();
          if (look.value && some_inexact<R / 4>(&a[0][0])) inexact = 1;
#pragma unroll
          for (int i = 0; i < R / 32; ++i) {
            const int k8 = wave_value((tid + i * kMThreads) / R);
#pragma unroll
            for (int j = 0; j < 8; ++j) a[i][j] = k8 / 2 * 4 + j / 2 < cnt ? a[i][j] : 0.f;
            const Split<h8> x = split_eight(a[i]);
            __bf16* to = L + tid % R * TS + k8 * 8;
            *(h8*)to = x.hi;
            *(h8*)(to + PL2) = x.mid;
            *(h8*)(to + 2 * PL2) = x.lo;
          }
          const bool small_cols = look.value && __ballot(some_inexact<32>(&b[0][0])) != 0ull;
          Split<h8> y[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) y[t] = split_eight(b[t]);
          __syncthreads();
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            f16v acc = TT_ZERO16;
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (4 * t < cnt)  // uniform: else no prefix of this step
                acc = mfma_split(split_from<PL2>(L + (mt * 32 + l32) * TS + 16 * t + 8 * half), y[t], acc);
            if (recheck(acc) || small_cols || inexact) {
              acc = TT_ZERO16;
              for (int k = half; k < 4 * cnt; k += 2)
                acc = mfma32(g1[(size_t)i1_of[k / 4] * S1 + (k % 4) * R + mt * 32 + l32],
                             dPsum[(size_t)q_of[k / 4] * PN + (k % 4) * W + col], acc);
            }
            sum[mt] += acc;
          }
          if (c + 1 == c1 || next.x != bin) {  // the group or the slice ends here
            float* dst = part2 + (size_t)first * S2;
            const uint32_t mine = 4 * half * W + col;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                (dst + (mt * 32 + 8 * (v / 4) + v % 4) * W)[mine] = sum[mt][v];
                sum[mt][v] = 0.f;
              }
            first = c + 1;
          }
          desc = next;
        }
      } else {
        const int c = c0 + sub - UN;
        if (c >= c1) continue;  // uniform for the block
        constexpr int NT = R / 32, MW = NT >= 4 ? 2 : 1;  // tiles of 32 lines of a wavefront
        // the thread number anew: nothing derived from it here is kept in registers across the dG2 units
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int w = tid / kWave, half = tid % kWave / 32, l32 = tid % 32;
        const int4 desc = c2_desc[c];
        const int cnt = desc.z;
        chunk_records(c, cnt);
        const float* Bm = g2 + (size_t)desc.x * S2;
        const int nt = w % NT, mt0 = w / NT;
        f4 ra[2], rb[R / 32];
        auto fetch = [&](int k0) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int e = tid + i * kMThreads, r = e / (KD / 4), k = e % (KD / 4) * 4;
            ra[i] = *(const f4*)(dPsum + (size_t)q_of[r / 4] * PN + (r % 4) * W + k0 + k);
          }
#pragma unroll
          for (int i = 0; i < R / 32; ++i) {
            const int e = tid + i * kMThreads, r = e / (KD / 4), k = e % (KD / 4) * 4;
            rb[i] = *(const f4*)(Bm + (size_t)r * W + k0 + k);
          }
        };
        f16v acc[MW];
#pragma unroll
        for (int x = 0; x < MW; ++x) acc[x] = TT_ZERO16;
        fetch(0);
#pragma unroll 1
        for (int k0 = 0; k0 < W; k0 += KD) {
          if (k0 > 0) __syncthreads();
          if (look.value && (some_inexact<8>((const float*)ra) || some_inexact<R / 8>((const float*)rb))) inexact = 1;
          auto put = [&](int line, int e, f4 v) {
            const Split<h4> x = split_four(v);
            __bf16* to = L + (line + e / (KD / 4)) * KS + e % (KD / 4) * 4;
            *(h4*)to = x.hi;
            *(h4*)(to + PL1) = x.mid;
            *(h4*)(to + 2 * PL1) = x.lo;
          };
#pragma unroll
          for (int i = 0; i < 2; ++i) put(0, tid + i * kMThreads, ra[i]);
#pragma unroll
          for (int i = 0; i < R / 32; ++i) put(64, tid + i * kMThreads, rb[i]);
          __syncthreads();
          if (k0 + KD < W) fetch(k0 + KD);  // in flight while this step is multiplied
          TT_LOADS_DONE();
#pragma unroll
          for (int t = 0; t < KD / 16; ++t) {
            const Split<h8> y = split_from<PL1>(L + (64 + nt * 32 + l32) * KS + 16 * t + 8 * half);
#pragma unroll
            for (int x = 0; x < MW; ++x)
              acc[x] = mfma_split(split_from<PL1>(L + ((mt0 + x) * 32 + l32) * KS + 16 * t + 8 * half), y, acc[x]);
          }
        }
#pragma unroll
        for (int x = 0; x < MW; ++x) {
          const int mt = mt0 + x;
          if (mt * 8 < cnt && (recheck(acc[x]) || inexact)) {
            const float* ar = dPsum + (size_t)q_of[mt * 8 + l32 / 4] * PN + (l32 % 4) * W + half * (W / 2);
            const float* br = Bm + (size_t)(nt * 32 + l32) * W + half * (W / 2);
            acc[x] = TT_ZERO16;
#pragma unroll 4
            for (int j = 0; j < W / 2; ++j) acc[x] = mfma32(ar[j], br[j], acc[x]);
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int ql = mt * 8 + 2 * (v / 4) + half;
            if (ql < cnt)
              dg1part[(size_t)q_of[ql] * S1 + (v % 4) * R + nt * 32 + l32] = acc[x][v];
          }
        }
      }
    }
  };
  if (ctr->small != 0) walk(std::true_type{});
  else walk(std::false_type{});
}

// ---------------------------------------------------------------------------------------------
// dPsum_q = sum over the unique ids u of prefix q of g_u G3[i3(u)]^T  (16 x D3 times D3 x R).
// One wavefront per prefix, or a block: its wavefronts take runs of MOST ids in turn, their sums meet in LDS and
// are added in their order.  by_block gives every prefix to a block; else each wavefront has one, and those of
// them with more than kLongIds ids are taken by all four afterwards.  The ids of a prefix extend the contraction
// index: 16 / D3 of them (a group) are one step, lane group kg holds four neighbours of a row of one id, so that a
// load instruction brings 16 bytes a lane and as many lines as it has to.
//
// A wavefront's long prefix is a chain of round trips that outlasts the kernel.  n = (400,400,2040), d = (4,4,8),
// rank 64, this kernel with every prefix left to its wavefront / as it is: 6,000 ids, 2,000 of them of one prefix,
// 444 / 119 us, 30,000 with 8 x 1,500 390 / 121, 40,000 with 300 x 60 75 / 75.  With 64 in place of 128, 200,000
// ids of n = (160,160,500) with 72 a prefix took 163 us instead of 156.
constexpr int kLongIds = 128;
template <int R, int D3, int MOST>
__device__ __forceinline__ void u_bwd_role(
    int block, int nblocks, bool by_block, f4 (*part)[R / 16][kWave], const float* __restrict__ g3,
    const float* __restrict__ grad, const float* __restrict__ gsum, const int* __restrict__ u_code,
    const int* __restrict__ u_i3, const int* __restrict__ q_us, float* __restrict__ dPsum,
    Counters* __restrict__ ctr) {
  constexpr int PN = 16 * R, S3 = R * D3, D = 16 * D3, NT = R / 16, KS = D3 / 4, IPG = 4 / KS;
  const int w = wave_value(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int l16 = lane % 16, kg = lane / 16;
  const int Q = ctr->Q, run = by_block ? 1 : kMWaves;  // prefixes of a block's turn
  for (int q0 = block * run; q0 < Q; q0 += nblocks * run) {
    int q = q0, u0 = 0, u1 = 0;
    uint32_t whole = 1u;  // prefixes of the turn that the whole block takes
    bool shared = by_block;
    if (!by_block) {
      int at[kMWaves + 1];  // one round trip, and none that waits for the last prefix's stores (scalar loads)
#pragma unroll
      for (int k = 0; k <= kMWaves; ++k) at[k] = q_us[min(q0 + k, Q)];
      whole = 0u;
#pragma unroll
      for (int k = 0; k < kMWaves; ++k) {
        whole |= at[k + 1] - at[k] > kLongIds ? 1u << k : 0u;
        u0 = w == k ? at[k] : u0;
        u1 = w == k ? at[k + 1] : u1;
      }
      q += w;
      if (u1 - u0 > kLongIds) u1 = u0;
    }
    for (;; shared = true) {
      if (shared) {
        if (whole == 0) break;
        q = q0 + __ffs((int)whole) - 1;
        whole &= whole - 1;
        u0 = wave_value(q_us[q]);
        u1 = wave_value(q_us[q + 1]);
      }
      if (u1 == u0) continue;
      f4 acc[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = f4{0.f, 0.f, 0.f, 0.f};
      const int first = u0 + (shared ? w * MOST : 0), hop = shared ? kMWaves * MOST : MOST;
      auto id_of = [&](int ub) { return min(ub + lane % MOST, u1 - 1); };
      int next_i3 = u_i3[id_of(first)], next_code = u_code[id_of(first)];
      for (int ub = first; ub < u1; ub += hop) {
        const int n = min(MOST, u1 - ub);
        const int myi3 = next_i3, mycode = next_code;
        next_i3 = u_i3[id_of(ub + hop)];  // on their way while this round's rows are
        next_code = u_code[id_of(ub + hop)];
        auto round = [&](auto groups, int i0) {
          constexpr int NG = decltype(groups)::value;
          f4 a[NG], b[NG][NT];
#pragma unroll
          for (int x = 0; x < NG; ++x) {
            const int i = min(i0 + x * IPG + kg / KS, n - 1);
            const float* gp = grad_row_ptr(__shfl(mycode, i), grad, gsum, D) + l16 * D3 + kg % KS * 4;
            const float* cp = g3 + (size_t)(uint32_t)__shfl(myi3, i) * S3 + l16 * D3 + kg % KS * 4;
            a[x] = *(const f4*)gp;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) b[x][nt] = *(const f4*)(cp + nt * 16 * D3);
          }
          TT_LOADS_DONE();
#pragma unroll
          for (int x = 0; x < NG; ++x) {
            // lanes without an id: both factors are zero, whatever the last one holds
            if (i0 + (x + 1) * IPG > n) {
              const bool on = i0 + x * IPG + kg / KS < n;
#pragma unroll
              for (int s = 0; s < 4; ++s) {
                a[x][s] = on ? a[x][s] : 0.f;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) b[x][nt][s] = on ? b[x][nt][s] : 0.f;
              }
            }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma16(a[x][s], b[x][nt][s], acc[nt]);
          }
        };
        if (MOST > IPG && n > MOST / 2) round(std::integral_constant<int, MOST / IPG>{}, 0);
        else
          for (int i0 = 0; i0 < n; i0 += IPG) round(std::integral_constant<int, 1>{}, i0);
      }
      if (shared) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) part[w][nt][lane] = acc[nt];
        __syncthreads();
        // wavefront w adds up and stores every kMWaves-th tile
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          if (nt % kMWaves == w) {
            f4 sum = part[0][nt][lane];
#pragma unroll
            for (int k = 1; k < kMWaves; ++k) sum += part[k][nt][lane];
            acc[nt] = sum;
          }
        __syncthreads();
      }
      float* dst = dPsum + (size_t)q * PN;
      bool inexact = false;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        if (!shared || nt % kMWaves == w) {
          inexact |= some_inexact<4>((const float*)&acc[nt]);
#pragma unroll
          for (int v = 0; v < 4; ++v) dst[(4 * kg + v) * R + nt * 16 + l16] = acc[nt][v];
        }
      if (__ballot(inexact) && lane == 0) atomicOr(&ctr->small, 1);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// part3[c]^T = sum over the <= 16 unique ids u of one by-i3 chunk of g_u^T P_q(u)
// (D3 x 16 times 16 x R; the D3 rows occupy the first rows of a 16-row tile), UB ids at a time.
template <int R, int D3, int UB>
__device__ __forceinline__ void dg3_chunk(
    int c, const float* __restrict__ P, const float* __restrict__ grad,
    const float* __restrict__ gsum, const int2* __restrict__ c3_item,
    const int4* __restrict__ c3_desc, float* __restrict__ part3) {
  constexpr int PN = 16 * R, S3 = R * D3, D = 16 * D3, NT = (R + 15) / 16;
  const int lane = threadIdx.x % kWave;
  const int l16 = lane % 16, kg = lane / 16;
  // rank 8: half of the 16 columns of the only tile exist; the others load column 0 and are dropped
  const bool col_on = R >= 16 || l16 < R;
  const int lcol = col_on ? l16 : 0;
  {
    const int2 item = c3_item[(size_t)c * kChunk3 + lane % kChunk3];
    const int cnt = c3_desc[c].z;
    // records past the chunk's count are unwritten; only lanes below cnt are ever read
    const int mycode = item.x, myq = item.y;
    f4 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = f4{0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < cnt; i0 += UB) {
      float a[UB][4], b[UB][NT][4];
#pragma unroll
      for (int x = 0; x < UB; ++x) {
        const int i = min(i0 + x, cnt - 1);
        const float* gp = grad_row_ptr(lane_value(mycode, i), grad, gsum, D) + (4 * kg) * D3 +
                          (l16 < D3 ? l16 : 0);
        const float* pp = P + (size_t)lane_value(myq, i) * PN + (4 * kg) * R + lcol;
#pragma unroll
        for (int s = 0; s < 4; ++s) a[x][s] = gp[s * D3];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int s = 0; s < 4; ++s) b[x][nt][s] = pp[s * R + nt * 16];
      }
      TT_LOADS_DONE();
#pragma unroll
      for (int x = 0; x < UB; ++x) {
        const bool on = (i0 + x < cnt) && (l16 < D3);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[nt] = mfma16(on ? a[x][s] : 0.f, b[x][nt][s], acc[nt]);
      }
    }
    float* dst = part3 + (size_t)c * S3;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j3 = 4 * kg + v;
        if (j3 < D3 && col_on) dst[(nt * 16 + l16) * D3 + j3] = acc[nt][v];
      }
  }
}

// ---------------------------------------------------------------------------------------------
// Sixteen 4 x 4 products, one term: tile b = lane/4, A[i] in lane i of the tile, B[j] in lane j, D[i][j] in
// accumulator i of lane j.  The four tiles of a run of sixteen lanes share the A of the run's tile FROM.
template <int FROM>
__device__ __forceinline__ f4 mfma_shared(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 2, FROM, 0);
}

// x of lanes l and l ^ 32 added up in the lower half of the lanes, y of both in the upper; the same for lanes l and
// l ^ 16: x in the lower sixteen lanes of a half, y in the upper.
__device__ __forceinline__ float add_halves(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                  false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float add_rows(float x, float y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                  false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// The same partial sum for ranks 64 and 128, where a prefix product is 4 to 8 KiB and the loads above would be 16 to
// 32 four-byte loads per id.  The contraction runs over the 16 rows m = 4*j1 + j2 of the product; lane group kg
// takes j2 = kg and the four j1, 16 bytes along a row: columns 64x + 4*l16 + t.  Products of 4 x 4, D3/4 of them
// over the height of g^T: 16 x 16 tiles would be half (D3 = 8) or three quarters (D3 = 4) empty.  The gradient row
// (16 x D3, row-major) is read with NL loads that together cover it contiguously: lane l16 = jj*D3 + j3 of group kg
// has g[4*(y*G + jj) + kg][j3], and the quad that holds four j3 of a row feeds all quads of its group.  The groups'
// sums are added up at the end, which leaves each with one column of four.
template <int R, int D3, int UB>
__device__ __forceinline__ void dg3_chunk_rows(
    int c, const float* __restrict__ P, const float* __restrict__ grad,
    const float* __restrict__ gsum, const int2* __restrict__ c3_item,
    const int4* __restrict__ c3_desc, float* __restrict__ part3) {
  constexpr int PN = 16 * R, S3 = R * D3, D = 16 * D3, NX = R / 64, JH = D3 / 4;
  constexpr int G = 16 / D3, NL = 4 / G;  // rows of g in sixteen lanes; loads per gradient row
  const int lane = threadIdx.x % kWave;
  const int l16 = lane % 16, kg = lane / 16;
  const int2 item = c3_item[(size_t)c * kChunk3 + lane % kChunk3];
  const int cnt = wave_value(c3_desc[c].z);
  // records past the chunk's count are unwritten; only lanes below cnt are ever read
  const int mycode = item.x, myq = item.y;
  f4 acc[NX][4][JH];
#pragma unroll
  for (int y = 0; y < NX; ++y)
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int jh = 0; jh < JH; ++jh) acc[y][t][jh] = f4{0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < cnt; i0 += UB) {
    float g[UB][NL];
    f4 b[UB][NX][4];
#pragma unroll
    for (int x = 0; x < UB; ++x) {
      const int i = min(i0 + x, cnt - 1);
      const float* gp = grad_row_ptr(lane_value(mycode, i), grad, gsum, D) + kg * D3 + l16 % D3;
      const float* pp = P + (size_t)lane_value(myq, i) * PN + kg * R + l16 * 4;
#pragma unroll
      for (int y = 0; y < NL; ++y) g[x][y] = gp[4 * (y * G + l16 / D3) * D3];
#pragma unroll
      for (int y = 0; y < NX; ++y)
#pragma unroll
        for (int j1 = 0; j1 < 4; ++j1) b[x][y][j1] = *(const f4*)(pp + y * 64 + j1 * (4 * R));
    }
    TT_LOADS_DONE();
#pragma unroll
    for (int x = 0; x < UB; ++x) {
      if (i0 + x >= cnt) break;  // uniform
      auto term = [&](auto row, auto height) {
        constexpr int j1 = decltype(row)::value, jh = decltype(height)::value;
        if constexpr (jh < JH) {
#pragma unroll
          for (int y = 0; y < NX; ++y)
#pragma unroll
            for (int t = 0; t < 4; ++t)
              acc[y][t][jh] = mfma_shared<j1 % G * JH + jh>(g[x][j1 / G], b[x][y][j1][t], acc[y][t][jh]);
        }
      };
      auto terms = [&](auto row) {
        term(row, std::integral_constant<int, 0>{});
        term(row, std::integral_constant<int, 1>{});
      };
      terms(std::integral_constant<int, 0>{});
      terms(std::integral_constant<int, 1>{});
      terms(std::integral_constant<int, 2>{});
      terms(std::integral_constant<int, 3>{});
    }
  }
  // group kg ends with t = 0, 2, 1, 3
  const int t = kg == 1 ? 2 : kg == 2 ? 1 : kg;
  float* dst = part3 + (size_t)c * S3 + (4 * l16 + t) * D3;
#pragma unroll
  for (int y = 0; y < NX; ++y)
#pragma unroll
    for (int jh = 0; jh < JH; ++jh) {
      f4 sum;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        sum[v] = add_rows(add_halves(acc[y][0][jh][v], acc[y][1][jh][v]), add_halves(acc[y][2][jh][v], acc[y][3][jh][v]));
      *(f4*)(dst + y * 64 * D3 + 4 * jh) = sum;
    }
}

// ---------------------------------------------------------------------------------------------
// The two gradient steps that only need the per-id gradient sums in one launch: dPsum per prefix, and the
// partial G3 gradients per by-i3 chunk.  The first is bound by its stores (a product per prefix) and the second by its
// gathers (one per id), so that the roles have half of the blocks each and alternate, eight blocks at a time, one to
// an XCD.  Few prefixes of many ids leave most wavefronts of the first role without one: there a block takes a prefix,
// and that role has as many blocks as prefixes and goes first: alternating, its blocks wait for compute units and are
// the kernel's end.  The line is a number of prefixes, and lower at d3 = 4, where rounds are shorter; fewer than
// kManyIds ids each leave wavefronts of the block without any.  This kernel in us, a wavefront / a block a prefix,
// n = (160,160,500):
//   d, rank, ids                  prefixes
//   (4,4,8),  64, 200,000           500: 130 / 124   2,000: 158 / 145   2,778: 157 / 153   4,167: 160 / 169
//   (4,4,8), 128, 100,000           250: 152 / 112   1,000: 166 / 127   2,083: 161 / 161   4,167: 155 / 183
//   (8,4,4),  64, 100,000 (slabs)   500:  75 /  66   1,000:  82 /  71   2,000: 101 / 104   2,778: 110 / 114
//   (8,4,4), 128,  50,000 (slabs)   250:  91 /  66     500:  79 /  67   1,000:  89 /  92   1,389: 101 / 107
// and with 2, 4, 8 and 16 ids to each of 2,000 prefixes, (4,4,8), rank 128: 16 / 23, 23 / 29, 35 / 41, 55 / 54.
// 500,000 Zipf ids of (480,500,500) x (8,4,4) at rank 128: 1272 alternating, 1490 one after the other.
constexpr int kManyIds = 16;  // ids per prefix of the batch

template <int R, int D3>
__global__ __launch_bounds__(kMThreads) void k_id_bwd_mfma(
    const float* __restrict__ g3, const float* __restrict__ P, const float* __restrict__ grad,
    const float* __restrict__ gsum, const int* __restrict__ u_code, const int* __restrict__ u_i3,
    const int* __restrict__ q_us, const int2* __restrict__ c3_item,
    const int4* __restrict__ c3_desc, float* __restrict__ dPsum, float* __restrict__ part3,
    Counters* __restrict__ ctr) {
  constexpr int kIds = 4;                  // ids of a wavefront's round (more: fewer wavefronts, 219 us against 207)
  constexpr int UB = R >= 128 ? 1 : 2;     // ids of a round of the other role (twice as many: rank 128 977 us a step,
                                           // against 967, at 100,000 uniform ids of 136^3 x (8,4,4))
  __shared__ f4 part[kMWaves][R / 16][kWave];
  constexpr int kFewPrefixes = D3 == 8 ? 3072 : 1024;
  const bool many = ctr->Q <= kFewPrefixes && ctr->U >= (int64_t)kManyIds * ctr->Q;
  const int b = blockIdx.x, half = gridDim.x / 2;  // a multiple of eight
  const int first = many ? min((ctr->Q + kXcds - 1) / kXcds * kXcds, half) : half;  // blocks of the first role
  const bool ids = many ? b < first : b / kXcds % 2 == 0;
  const int block = many ? (ids ? b : b - first) : b / (2 * kXcds) * kXcds + b % kXcds;
  if (ids) {
    u_bwd_role<R, D3, kIds>(block, first, many, part, g3, grad, gsum, u_code, u_i3, q_us, dPsum, ctr);
  } else {
    const int nchunk = ctr->nchunk3;
    for (int c = block * kMWaves + (int)threadIdx.x / kWave; c < nchunk; c += ((int)gridDim.x - first) * kMWaves)
      dg3_chunk_rows<R, D3, UB>(c, P, grad, gsum, c3_item, c3_desc, part3);
  }
}

// ---------------------------------------------------------------------------------------------
// Ranks up to 32: the whole middle of the backward pass in one launch, without dPsum ever leaving
// the chip.  A block owns one by-i2 chunk (<= 16 prefixes q, Bm = G2[i2]):
//   (i)   dPsum_q = sum over the ids u of q of g_u G3[i3(u)]^T; results go to an LDS tile of 64 rows
//         (row = 4*prefix + j1) by 4R columns, Bm is put into LDS beside it
//   (ii)  wavefronts 0..3: dg1part[q] = dPsum_q Bm^T for four prefixes each (operands from LDS)
//   (iii) other wavefronts: 32 columns each of part2[c] = sum_q G1[i1(q)]^T dPsum_q
// Blocks past the chunk range take the by-i3 chunks of the G3 gradient (dg3_role), one per
// wavefront; that step only needs the per-id gradient sums and the cached prefix products, so
// both run side by side.
//
// (i) is bound by round trips to memory: a wavefront takes 16 / WAVES prefixes, SO ids in flight, and its
// longest prefix sets the time.  With skewed ids one prefix of a chunk has hundreds of ids and the others a
// few, so the long ones are taken first by the whole block, one after the other, WAVES * SC ids in flight;
// the wavefronts' sums meet in LDS and are added in their order.  Which are long is the choice that takes
// the fewest rounds, a long one counted with its barriers and, where it loads twice the ids, as two (at one
// each, 60,000 clustered ids of 136^3, d = (8,4,4), rank 16 took 79 us, and 500,000 of (480,480,482) 275).
// The kernel with every prefix left to its wavefront / now, us; Zipf: hot ids together, as in tables renumbered by
// partition.
//   n, d, rank, ids                          Zipf        clustered   uniform
//   (480,480,482), (4,4,8), 16, 500,000      310 /  92   210 / 126   241 / 241
//   (480,480,482), (4,4,8), 32, 500,000      285 / 191   196 / 147   474 / 470
//   (480,480,482), (8,4,4), 16, 500,000      376 / 173   278 / 230   420 / 416
//   (136,136,136), (4,4,8), 32, 200,000       85 /  57    80 /  81   117 / 116
//   (136,136,136), (8,4,4), 16,  60,000       80 /  40    69 /  60    49 /  49
//   (55,55,56),    (8,4,4), 16,  50,000       48 /  34    41 /  30    32 /  30
// The chunk's records wait in LDS for the steps behind (i): in registers they made the form of rank 32 and d3 = 8
// spill four (uniform ids of the second line 507 us).
//
// WAVES: eight.  Four at ranks up to 16 where the batch has fewer than four ids per prefix of the table: a
// round then is mostly one or two ids a prefix, and two blocks of four hold twice the prefixes (uniform ids
// of (480,480,482), eight / four wavefronts: 268 / 243 us at 500,000 ids and d = (4,4,8), 170 / 137 at 300,000
// and (4,4,4); with 37 ids a prefix, n = (40,40,500), 27 / 33).  The line is one for all ids: at 13 items a
// prefix, 250,000 ids of 136^3 with d = (8,4,4), rank 16, clustered ones take 93 / 110, Zipf ones 52 / 49.
// Blocks past the by-i2 chunk range take the by-i3 chunks of the G3 gradient, one per wavefront, which gather a
// prefix product per id.  A group's chunks are in prefix order: workgroups go to the eight XCDs round robin, and
// XCD x takes the x-th eighth of every group and walks the eighths of all groups side by side, so that the
// products it gathers at one time are few, and its own.  A group is a column, or several where its eighth is longer
// than walk_steps (twice the mean, or the longest eighth if that is less): its chunks go to its columns in turn, so
// that it keeps pace with the others and no wavefront waits for the one group that is left.  Steps in us with an
// eighth of all chunks in index order / side by side, one column a group / as it is:
//   200,000 ids of 136^3, rank 32, one group with 2.5 / 10 / 35 times the mean: 249 / 228 / 228, 260 / 245 / -,
//     261 / 256 / -; look-ahead 214 / 196 / 197, 225 / 214 / 208, 226 / 224 / 214 (a list of the chunks by prefix, 4 to
//     6 us of the index pipeline: 203, 215, 220)
//   500,000 of 480x480x482, rank 16, the same: 478 / 471 / 472, 481 / 477 / -, 498 / 525 / -; look-ahead 450 / 443 /
//     445, 453 / 451 / 449, 472 / 496 / 466
//   Zipf ids, whose groups are alike: 172 -> 169 and 376.1 -> 375.6 from index order; look-ahead 122 and 330 either way
// Columns of one mean instead of two: 500,000 uniform ids of 480x480x482 471 -> 480 us, the unequal groups 1 % less.
// Where groups have few chunks, places without one cost more than neighbours bring (index order / side by side, uniform
// ids): 120x120x500, rank 32, 2 / 6 / 10 / 16 / 24 chunks a group 91 / 96, 108 / 110, 120 / 121, 137 / 135, 160 / 152;
// (60,60,2000) x (8,4,4), rank 16, 6 / 12 / 16 chunks 113 / 118, 152 / 157, 172 / 176.
template <class F>
__device__ __forceinline__ void walk_chunks3(int xcd, int wave, int nwaves, const int4* __restrict__ walk3,
                                             const Counters* __restrict__ ctr, F take) {
  const int chunks = ctr->nchunk3, cols = ctr->walk_cols;
  const int lo = (int)((int64_t)chunks * xcd / kXcds), hi = (int)((int64_t)chunks * (xcd + 1) / kXcds);
  const int n = cols > 0 ? ctr->walk_steps * cols : hi - lo;
  for (int i = wave; i < n; i += nwaves) {
    int c = lo + i, end = hi;
    if (cols > 0) {
      const int j = (int)((uint32_t)i / (uint32_t)cols);
      const int4 col = walk3[i - j * cols];
      c = col.x + col.y * xcd / kXcds + j * col.w + col.z;
      end = col.x + col.y * (xcd + 1) / kXcds;
    }
    if (c < end) take(c);
  }
}

template <int R, int D3, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, 6) void k_bwd_mid_mfma(
    const float* __restrict__ g1, const float* __restrict__ g2, const float* __restrict__ g3,
    const float* __restrict__ P, const float* __restrict__ grad, const float* __restrict__ gsum,
    const int* __restrict__ u_code, const int* __restrict__ u_i3, const int4* __restrict__ c2_item,
    const int4* __restrict__ c2_desc, const int2* __restrict__ c3_item,
    const int4* __restrict__ c3_desc, const int4* __restrict__ walk3,
    float* __restrict__ dg1part, float* __restrict__ part2, float* __restrict__ part3,
    int chunk_blocks, const Counters* __restrict__ ctr) {
  static_assert(R == 8 || R == 16 || R == 32, "the LDS tiles are sized for ranks up to 32");
  constexpr int W = 4 * R, S1 = 4 * R, S2 = R * W, S3 = R * D3, D = 16 * D3;
  constexpr int TS = W + 4;  // padded row stride of the LDS tiles (keeps 16-byte alignment)
  constexpr int NT16 = (R + 15) / 16, KS = D3 / 4;
  constexpr int kMidThreads = WAVES * kWave, kParts = WAVES * NT16 * 256;
  __shared__ int q_of[kChunk2], i1_of[kChunk2];  // records of the chunk's prefixes for the steps behind (i)
  __shared__ __align__(16) float T[64 * TS];
  __shared__ __align__(16) float Bl[R * TS > kParts ? R * TS : kParts];  // wavefronts' sums of a long prefix, then Bm
  const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
  if ((int)blockIdx.x >= chunk_blocks) {
    const int rel = (int)blockIdx.x - chunk_blocks;
    walk_chunks3((int)blockIdx.x % kXcds, rel / kXcds * WAVES + w, ((int)gridDim.x - chunk_blocks) / kXcds * WAVES,
                 walk3, ctr, [&](int c) { dg3_chunk<R, D3, 4>(c, P, grad, gsum, c3_item, c3_desc, part3); });
    return;
  }
  // records, descriptor and chunk count are read together (the grid never exceeds the tables)
  const int c = blockIdx.x;
  const int l16 = lane % 16, kg = lane / 16;
  int4 item = c2_item[(size_t)c * kChunk2 + l16];
  const int4 desc = c2_desc[c];
  if (c >= ctr->nchunk2) return;
  if (l16 >= desc.z) item = int4{-1, 0, 0, 0};  // records past the chunk's count are unwritten
  if (tid < kChunk2) {
    q_of[tid] = item.x;
    i1_of[tid] = item.y;
  }
  // Bm is needed behind the barrier only: below rank 32 its words wait in registers, at rank 32 they are
  // loaded behind (i), where registers are free
  const f4* Bm = (const f4*)(g2 + (size_t)desc.x * S2);
  constexpr int NB = (R * W / 4 + kMidThreads - 1) / kMidThreads;
  f4 bm[NB];
  auto load_bm = [&] {
#pragma unroll
    for (int k = 0; k < NB; ++k) bm[k] = Bm[min(tid + k * kMidThreads, R * W / 4 - 1)];
  };
  if constexpr (R < 32) load_bm();
  // rank 8: rows / columns 8..15 of the only 16-wide tile do not exist; such lanes read row 0 and
  // their results are dropped
  const bool rank_on = R >= 16 || l16 < R;
  const int lrow = rank_on ? l16 : 0;
  // (i): SC ids of a long prefix in flight together, SO of the others (what 80 registers hold; eight
  // wavefronts of two prefixes take two ids of each where rows are 128 floats).  Lane x holds where the
  // gradient row and the G3 slice of the round's id x are.
  constexpr int SC = R <= 16 && KS == 1 ? 16 : 8, SO = WAVES == 4 || R == 32 || KS == 1 ? 8 : 4;
  constexpr int kBarriers = KS == 2 ? 1 : R <= 16 ? 4 : 2;
  constexpr bool kAhead = R < 32 || KS == 1;  // registers for the next round's codes
  auto load_ids = [&](int mycode, int myi3, auto& a, auto& b) {
#pragma unroll
    for (int sl = 0; sl < (int)(sizeof(a) / sizeof(a[0])); ++sl) {
      const float* gp = grad_row_ptr(lane_value(mycode, sl), grad, gsum, D) + l16 * D3 + KS * kg;
      const float* cp = g3 + (size_t)lane_value(myi3, sl) * S3 + lrow * D3 + KS * kg;
#pragma unroll
      for (int k = 0; k < KS; ++k) a[sl][k] = gp[k];
#pragma unroll
      for (int nt = 0; nt < NT16; ++nt)
#pragma unroll
        for (int k = 0; k < KS; ++k) b[sl][nt][k] = cp[nt * 16 * D3 + k];
    }
    TT_LOADS_DONE();
  };
  // accumulator element v of lane (kg, l16) is dPsum_q[m = 4*kg + v][n = nt*16 + l16], i.e. row
  // j1 = kg of the prefix and column j2*R + n with j2 = v
  auto put_sum = [&](int p, const f4 (&sum)[NT16]) {
#pragma unroll
    for (int nt = 0; nt < NT16; ++nt)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (rank_on) T[(p * 4 + kg) * TS + v * R + nt * 16 + l16] = sum[nt][v];
  };
  int ids = item.w - item.z;
  uint32_t longs = 0;  // prefixes taken by the whole block
  if (__ballot(ids > 16)) {
    constexpr int UB = SO * WAVES / 16;
    // rounds in all if the prefixes with more ids than this lane's are long; kBarriers stands for the barriers and,
    // where SC is twice SO, for the longer rounds
    const int mine = (ids + SC * WAVES - 1) / (SC * WAVES) + kBarriers;
    int cost = (ids + UB - 1) / UB;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (lane_value(ids, k) > ids) cost += lane_value(mine, k);
    int least = cost;
#pragma unroll
    for (int o = 1; o < 16; o *= 2) least = min(least, __shfl_xor(least, o));
    const int limit = lane_value(ids, __ffsll((long long)__ballot(cost == least)) - 1);
    longs = (uint32_t)__ballot(ids > limit) & 0xffffu;
  }
  for (uint32_t left = longs; left; left &= left - 1) {
    const int p = __ffs((int)left) - 1;
    const int n = lane_value(ids, p), u0 = lane_value(item.z, p);
    f4 acc[NT16];
#pragma unroll
    for (int nt = 0; nt < NT16; ++nt) acc[nt] = f4{0.f, 0.f, 0.f, 0.f};
    auto id_of = [&](int i0) { return u0 + min(i0 + lane % SC, n - 1); };
    int mycode = 0, myi3 = 0;
    if (kAhead) {
      mycode = u_code[id_of(w * SC)];
      myi3 = u_i3[id_of(w * SC)];
    }
    for (int i0 = w * SC; i0 < n; i0 += WAVES * SC) {
      const int at = id_of(kAhead ? i0 + WAVES * SC : i0);
      const int next_code = u_code[at], next_i3 = u_i3[at];
      if (!kAhead) {
        mycode = next_code;
        myi3 = next_i3;
      }
      float a[SC][KS], b[SC][NT16][KS];
      load_ids(mycode, myi3, a, b);
#pragma unroll
      for (int sl = 0; sl < SC; ++sl)
        if (i0 + sl < n) {
#pragma unroll
          for (int nt = 0; nt < NT16; ++nt)
#pragma unroll
            for (int k = 0; k < KS; ++k) acc[nt] = mfma16(a[sl][k], b[sl][nt][k], acc[nt]);
        }
      if (kAhead) {
        mycode = next_code;
        myi3 = next_i3;
      }
    }
    f4* part = (f4*)Bl;
#pragma unroll
    for (int nt = 0; nt < NT16; ++nt) part[(w * NT16 + nt) * kWave + lane] = acc[nt];
    __syncthreads();
    if (p % WAVES == w) {
#pragma unroll
      for (int nt = 0; nt < NT16; ++nt) {
        f4 sum = part[nt * kWave + lane];
#pragma unroll
        for (int k = 1; k < WAVES; ++k) sum += part[(k * NT16 + nt) * kWave + lane];
        acc[nt] = sum;
      }
      put_sum(p, acc);
    }
    __syncthreads();
  }
  {
    constexpr int G = 16 / WAVES, UB = SO / G;
    if ((longs >> l16) & 1) ids = 0;
    f4 acc[G][NT16];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int nt = 0; nt < NT16; ++nt) acc[g][nt] = f4{0.f, 0.f, 0.f, 0.f};
    int most = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) most = max(most, lane_value(ids, G * w + g));
    const int myp = G * w + (lane % SO) / UB;  // the prefix of this lane's slot
    const int myu0 = __shfl(item.z, myp), myn = __shfl(ids, myp);
    const int rounds = (most + UB - 1) / UB;
    // the next round's codes are on their way while this round's rows are
    auto slot_on = [&](int r) { return r * UB + lane % UB < myn && lane < SO; };
    auto id_of = [&](int r) { return slot_on(r) ? myu0 + r * UB + lane % UB : 0; };
    int mycode = 0, myi3 = 0;
    if (kAhead) {
      mycode = u_code[id_of(0)];
      myi3 = u_i3[id_of(0)];
    }
    for (int r = 0; r < rounds; ++r) {
      const unsigned long long on_mask = __ballot(slot_on(r));
      const int at = id_of(kAhead ? r + 1 : r);
      const int next_code = u_code[at], next_i3 = u_i3[at];
      if (!kAhead) {
        mycode = next_code;
        myi3 = next_i3;
      }
      float a[SO][KS], b[SO][NT16][KS];
      load_ids(mycode, myi3, a, b);
#pragma unroll
      for (int sl = 0; sl < SO; ++sl) {
        // wavefront-uniform: empty slots cost no matrix-core time
        if ((on_mask >> sl) & 1ull) {
#pragma unroll
          for (int nt = 0; nt < NT16; ++nt)
#pragma unroll
            for (int k = 0; k < KS; ++k)
              acc[sl / UB][nt] = mfma16(a[sl][k], b[sl][nt][k], acc[sl / UB][nt]);
        }
      }
      if (kAhead) {
        mycode = next_code;
        myi3 = next_i3;
      }
    }
    if constexpr (R >= 32) load_bm();
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (!((longs >> (G * w + g)) & 1)) put_sum(G * w + g, acc[g]);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int i = tid + k * kMidThreads;
      if (R * W / 4 % kMidThreads == 0 || i < R * W / 4) *(f4*)&Bl[((i * 4) / W) * TS + (i * 4) % W] = bm[k];
    }
  }
  __syncthreads();

  if (w < 4) {
    // (ii) tile rows 16w .. 16w+15 (prefixes 4w .. 4w+3) times Bm^T, 16 x 16 output tiles; lane
    // group kg contracts over columns [KQ*kg, KQ*kg + KQ)
    constexpr int KQ = W / 4;
    const f4* arow = (const f4*)&T[(16 * w + l16) * TS + KQ * kg];
    f4 acc[NT16];
#pragma unroll
    for (int nt = 0; nt < NT16; ++nt) acc[nt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < KQ / 4; ++j) {
      const f4 x = arow[j];
#pragma unroll
      for (int nt = 0; nt < NT16; ++nt) {
        const f4 y = *(const f4*)&Bl[(16 * nt + lrow) * TS + KQ * kg + 4 * j];
        acc[nt] = mfma16(x.x, y.x, acc[nt]);
        acc[nt] = mfma16(x.y, y.y, acc[nt]);
        acc[nt] = mfma16(x.z, y.z, acc[nt]);
        acc[nt] = mfma16(x.w, y.w, acc[nt]);
      }
    }
    // accumulator element v: tile row 4*kg + v = prefix 4w + kg, j1 = v; column n = 16*nt + l16
    const int qv = q_of[4 * w + kg];
    if (qv >= 0) {
#pragma unroll
      for (int nt = 0; nt < NT16; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (rank_on) dg1part[(size_t)qv * S1 + v * R + 16 * nt + l16] = acc[nt][v];
    }
  }
  const int w3 = WAVES == 8 ? w - 4 : w;
  if (w3 >= 0 && w3 < W / 32) {
    // (iii) G1 rows of the sixteen prefixes (as the contraction index) times 32 columns of the tile
    const int half = lane / 32, l32 = lane % 32;
    float a[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      const int ql = 8 * half + j / 4;
      a[j] = g1[(size_t)i1_of[ql] * S1 + (j % 4) * R + (l32 < R ? l32 : 0)];
    }
    TT_LOADS_DONE();
#pragma unroll
    for (int j = 0; j < 32; ++j)
      if (q_of[8 * half + j / 4] < 0 || l32 >= R) a[j] = 0.f;
    const int n = w3 * 32 + l32;
    f16v acc = TT_ZERO16;
#pragma unroll
    for (int j = 0; j < 32; ++j) acc = mfma32(a[j], T[(32 * half + j) * TS + n], acc);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int mrow = 8 * (v / 4) + 4 * half + (v % 4);
      if (mrow < R) part2[(size_t)c * S2 + (size_t)mrow * W + n] = acc[v];
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Rows: one wavefront per tile of TSL sorted slots.  The distinct ids of a tile are taken in groups
// of up to 16/D3 consecutive ids that share a prefix: E^T = (their G3 slices, transposed, one below the
// other: 16 x R) times P_q^T (R x 16).  A lane's four accumulators are then four neighbours of a row, and
// one 16-byte store a lane writes whole rows of the group's ids; ids with several positions repeat it.
// Rows are written with non-temporal stores: nothing on this path reads them back.
//
// Operands are loaded as they lie in memory: P_q by whole lines into LDS, slices of G3 in 4 x 4 blocks that
// quads of lanes turn; those of the next group are in flight while a group is formed and stored.  Read as
// the matrix cores want them, each 16 bytes of P_q are a line of their own (64 cycles a load instruction)
// and G3 takes a load per element.  With those, and rows through LDS, the kernel took (500,000 ids of n =
// (480,480,482), d = (4,4,8), Zipf / clustered) 135 / 112 us at rank 64 and 58 / 54 at rank 16, now 96 / 95
// and 56 / 48; rank 128, 200,000 Zipf ids of (480,500,500) x (8,4,4): 276 -> 138.  At rank 32 and 200,000
// Zipf ids it is at the rate of random 512-byte stores (27 -> 26 us).
// Slots of a tile: short ones for short chains of groups (200,000 Zipf ids at rank 32: 26 / 30 / 38 us with
// 8 / 16 / 32), longer ones where a product is 4 to 8 KiB and neighbours share it (clustered ids at rank
// 64: 106 / 95 / 92 us; Zipf 98 / 96 / 105), and for large batches of 64-float rows, four ids a group: 8 / 16
// slots, 400,000 items of (272,136,136) 35.9 / 34.0 us Zipf ids at rank 16, 59.3 / 53.8 uniform at 32; 1,000,000
// clustered ones of (960,480,482) 64.8 / 51.0 at 16, 85.6 / 68.5 at 32; 1,000,000 Zipf ones 79.0 / 69.3 at 8.
// (Up to 131,072 rows 8: 100,000 uniform ids of 136^3 15.2 / 14.7, Zipf 15.4 / 15.9, 20,000 10.7 / 13.7.)
// Where the index kernels of a coming batch run beside this one, four times the wavefronts take the compute
// units from them (look-ahead steps in us, each loop a process of its own):
//   ids, n, rank                                8 / 16 / 32 slots
//   500,000 Zipf, (480,480,482), 16              - / 345 / 336
//   500,000 Zipf, (480,480,482), 8               - / 272 / 264
//   500,000 Zipf, (136,136,136), 32              - / 266 / 259
//   250,000 Zipf, (480,480,482), 8             171 / 165 / 162
//   200,000 Zipf, (480,480,482), 8             144 / 141 / 140
//   200,000 Zipf, hot ids together, the same   177 / 184 / 199
//   200,000 Zipf, (136,136,136), 32            140 / 140 / 143
//   140,000 Zipf, (480,480,482), 32            247 / 251 / 255
constexpr int kRowsSome = 1 << 17, kRowsMany = 1 << 18;
__host__ constexpr int row_slots(int R, int D3, bool beside, int B) {
  if (R > 32) return 16;
  if (beside && B > kRowsMany) return 32;
  return B > kRowsSome && (D3 == 4 || (beside && R <= 16)) ? 16 : 8;
}

template <int R, int D3, int TSL>
__global__ __launch_bounds__(kMThreads) void k_row_fwd_mfma(
    int B, const float* __restrict__ g3, const float* __restrict__ P,
    const int4* __restrict__ s_rec, float* __restrict__ out, Counters* ctr) {
  constexpr int PN = 16 * R, S3 = R * D3, D = 16 * D3, UPT = 16 / D3, KQ = R / 4;
  constexpr int RS = R + 4;                       // stride of a line of P in LDS
  constexpr int NP = (PN + 255) / 256;            // 16-byte words of P a lane loads
  constexpr int NC = R >= 16 ? R / 16 : 0;        // blocks of G3 a quad loads (rank 8: element by element)
  __shared__ __align__(16) float Pl[kMWaves][16 * RS];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int l16 = lane % 16, kg = lane / 16;
  const int ul = l16 / D3, j3 = l16 % D3;         // this lane's line of E^T as an operand
  const int my_id = kg * 4 / D3, my_j3 = kg * 4 % D3;  // and what its accumulators hold
  float* Pw = Pl[w];
  const int tile = blockIdx.x * kMWaves + w;
  if (tile * TSL >= B) return;
  const int s = lane < TSL ? tile * TSL + lane : B;
  const int4 rec = s_rec[min(s, B - 1)];  // {unique-id index, batch position, prefix, i3}
  const int mysu = s < B ? rec.x : -2;    // lanes past the batch: neither an id nor an out-of-range slot
  const uint32_t myb = (uint32_t)rec.y;
  if (s < B && myb >= (uint32_t)B) atomicOr(&ctr->err, 4);
  // out-of-range ids (the tail of the sorted order) get zero rows
  unsigned long long zero_slots = __ballot(mysu == -1 && myb < (uint32_t)B);
  while (zero_slots) {
    const int sl = __ffsll((long long)zero_slots) - 1;
    zero_slots &= zero_slots - 1;
    float* o = out + (size_t)(uint32_t)lane_value((int)myb, sl) * D;
    for (int e = lane; e < D; e += kWave) o[e] = 0.f;
  }
  const int nv = __popcll(__ballot(mysu >= 0));
  if (nv == 0) return;
  const int u_lo = lane_value(mysu, 0), nu = lane_value(mysu, nv - 1) - u_lo + 1;
  // lane e takes the tile's e-th distinct id: its first slot, prefix and i3
  const int su_before = __shfl_up(mysu, 1);
  const bool first = lane < nv && (lane == 0 || mysu != su_before);
  const int rank = lane < nv ? mysu - u_lo : nu - 1;
  const int to = (first ? rank : nu + lane - rank - 1) * 4;
  const int u_slot = __builtin_amdgcn_ds_permute(to, lane);
  const int myq = __builtin_amdgcn_ds_permute(to, rec.z), myi3 = __builtin_amdgcn_ds_permute(to, rec.w);
  // groups: every UPT-th id of a run of ids with one prefix starts one
  const int q_before = __shfl_up(myq, 1);
  const unsigned long long runs = __ballot(lane < nu && (lane == 0 || myq != q_before));
  const unsigned long long upto = runs & (lane == 63 ? ~0ull : ((2ull << lane) - 1ull));
  const int run_first = 63 - __clzll((long long)(upto | 1ull));
  const unsigned long long groups = __ballot(lane < nu && ((lane - run_first) % UPT) == 0);
  auto end_of = [&](int st) {
    const unsigned long long after = groups & ~((2ull << st) - 1ull);
    return after ? __ffsll((long long)after) - 1 : nu;
  };
  f4 p[NP], cv[NC > 0 ? NC : 1];
  float ce[NC > 0 ? 1 : KQ];
  int have = -1;  // prefix of p
  auto fetch = [&](int st) {
    const int q = lane_value(myq, st);
    if (q != have) {
      have = q;
      const f4* src = (const f4*)(P + (size_t)q * PN);
#pragma unroll
      for (int k = 0; k < NP; ++k) p[k] = src[PN < 256 ? lane % (PN / 4) : lane + k * kWave];
    }
    const float* C = g3 + (size_t)__shfl(myi3, min(st + ul, end_of(st) - 1)) * S3 + (KQ * kg) * D3;
    if constexpr (NC > 0) {
#pragma unroll
      for (int j = 0; j < NC; ++j) cv[j] = *(const f4*)(C + (4 * j + j3 % 4) * D3 + j3 / 4 * 4);
    } else {
#pragma unroll
      for (int j = 0; j < KQ; ++j) ce[j] = C[j * D3 + j3];
    }
  };
  fetch(0);
  int in_lds = -1;  // prefix whose product is in LDS
  for (int st = 0; st < nu;) {
    const int end = end_of(st);
    if (have != in_lds) {
      in_lds = have;
      wave_sync();
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int e = 4 * (lane + k * kWave);
        if (PN >= 256 || e < PN) *(f4*)(Pw + (e / R) * RS + e % R) = p[k];
      }
      wave_sync();
    }
    float c[KQ];
    if constexpr (NC > 0) {
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const f4 t = quad_turned(cv[j], lane);
        c[4 * j] = t.x;
        c[4 * j + 1] = t.y;
        c[4 * j + 2] = t.z;
        c[4 * j + 3] = t.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < KQ; ++j) c[j] = ce[j];
    }
    if (end < nu) fetch(end);  // in flight while this group is formed and stored
    const float* pr = Pw + l16 * RS + KQ * kg;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    if constexpr (KQ % 4 == 0) {
#pragma unroll
      for (int j = 0; j < KQ; j += 4) {
        const f4 v = *(const f4*)(pr + j);
        acc = mfma16(c[j], v.x, acc);
        acc = mfma16(c[j + 1], v.y, acc);
        acc = mfma16(c[j + 2], v.z, acc);
        acc = mfma16(c[j + 3], v.w, acc);
      }
    } else {
#pragma unroll
      for (int j = 0; j < KQ; ++j) acc = mfma16(c[j], pr[j], acc);
    }
    // A group of fewer than UPT ids holds its last one several times over: those lanes share its positions
    const int last = end - 1 - st, part = max(my_id - last, 0), parts = my_id >= last ? UPT - last : 1;
    const int id = st + min(my_id, last);
    const int s0 = __shfl(u_slot, id) + part, after = __shfl(u_slot, min(id + 1, nu - 1));
    const int s1 = id + 1 < nu ? after : nv;
    float* o = out + (size_t)l16 * D3 + my_j3;
    for (int at = s0; __ballot(at < s1) != 0ull; at += 4 * parts) {
      uint32_t b[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) b[k] = (uint32_t)__shfl((int)myb, min(at + k * parts, 63));
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (at + k * parts < s1 && b[k] < (uint32_t)B)
          __builtin_nontemporal_store(acc, (f4*)(o + (size_t)b[k] * D));
    }
    st = end;
  }
}

// ---------------------------------------------------------------------------------------------
// Sums grad_out over runs of equal ids (rows of D = 64*VPL floats, VPL floats per lane).
// A block takes 1024 consecutive sorted slots, 64 per wavefront.  Each wavefront loads the rows of
// its slots (32 at a time, all loads in flight together), adds them up run by run in slot order,
// and finishes the runs that lie inside its 64 slots; ids that occur once are skipped, later
// kernels read their row from grad_out directly.  Pieces of runs that cross wavefronts are joined
// in LDS.  No run crosses a block: the index pipeline cuts long runs of one id into entries at
// every multiple of kEntrySlots slots, which is the block size here.
// A wavefront with at most sparse_slots slots to load goes from one of them to the next instead of
// looking at all 64: with uniform ids the looking was the time (28 -> 8.4 us at 500,000 ids of 111 million
// rows, 16 -> 6 at 200,000 of 2.4 million, 18 -> 14.4 at 60,000 of 175,616).  Where the line lies, us with 32 /
// 48 slots: rows of 64 floats, 60,000 clustered ids 16.6 / 19.7 (18.4 where all look at all slots), 500,000
// 50.9 / 53.3 (57.4); ragged rows, which take more instructions a slot, 200,000 uniform ids of 56^3 with 100
// floats 30.9 / 34.8 (30.9); rows of 128 floats, 60,000 clustered ids 21.4 / 20.2 (21.5), 500,000 52.8 / 49.4
// (53.5).
// Rows of 64 floats go 8 at a time: rounds of 16 take 92 scalar registers, and one block less fits a compute
// unit: 520,000 uniform items 42 -> 33 us, 1,000,000 clustered ones 67 -> 51.
constexpr int kGsumWaves = 16;
constexpr int kGsumThreads = kGsumWaves * kWave;
constexpr int kGsumBlockSlots = kGsumWaves * kWave;  // 1024
constexpr int sparse_slots(int vpl, bool ragged) { return vpl == 2 && !ragged ? 48 : 32; }
static_assert(kGsumBlockSlots == kEntrySlots, "a block must own exactly one entry span");

template <int VPL>
struct LaneVec {
  float v[VPL];
};

// RAGGED: rows of Drt <= 64*VPL floats (any length), read with plain dword loads (their starts need not
// be 8-byte aligned).
template <int VPL, bool RAGGED>
__global__ __launch_bounds__(kGsumThreads) void k_gsum_block(int B, int Drt,
                                                          const float* __restrict__ grad,
                                                          const int* __restrict__ s_u,
                                                          const uint32_t* __restrict__ perm,
                                                          float* __restrict__ gsum, Counters* ctr) {
  constexpr int DP = kWave * VPL;          // padded row length
  const int D = RAGGED ? Drt : DP;
  constexpr int kRows = VPL <= 2 ? 32 : 64 / VPL;  // rows a wavefront has in flight (64 registers)
  __shared__ float part[kGsumWaves][2][DP];  // [wave][0 = head piece, 1 = tail piece]
  __shared__ int head_state[kGsumWaves];    // 0 none, 1 head piece ends in this wave, 2 it runs through
  __shared__ int tail_u[kGsumWaves];        // id whose run starts in this wave and continues, or -1
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int nbt = (B + kGsumBlockSlots - 1) / kGsumBlockSlots;
  for (int bt = blockIdx.x; bt < nbt; bt += gridDim.x) {
    const int wt0 = bt * kGsumBlockSlots + w * kWave;
    const int s = wt0 + lane;
    const int mysu = s < B ? s_u[s] : -1;
    const uint32_t myb = s < B ? perm[s] : 0u;
    if (s < B && myb >= (uint32_t)B) atomicOr(&ctr->err, 8);
    const int prev_su = (wt0 > 0 && wt0 - 1 < B) ? s_u[wt0 - 1] : -2;
    const int next_su = (wt0 + kWave < B) ? s_u[wt0 + kWave] : -2;
    const int nv = __popcll(__ballot(mysu >= 0));
    // a slot needs its row loaded unless its id occurs exactly once in the whole batch
    int su_before = __shfl_up(mysu, 1), su_after = __shfl_down(mysu, 1);
    if (lane == 0) su_before = prev_su;
    if (lane == kWave - 1) su_after = next_su;
    const bool need = mysu >= 0 && myb < (uint32_t)B && (su_before == mysu || su_after == mysu);
    const unsigned long long need_mask = __ballot(need);

    if (lane == 0) {
      head_state[w] = 0;
      tail_u[w] = -1;
    }
    LaneVec<VPL> acc;
    int cur = -2, cur_first = 0;
    auto flush = [&](int end_slot) {  // the run of cur covers tile slots [cur_first, end_slot)
      if (cur < 0) return;
      const bool starts_here = cur_first > 0 || prev_su != cur;
      const bool ends_here = end_slot < kWave || next_su != cur;
      if (starts_here && ends_here) {
        if (end_slot - cur_first > 1) {
          float* o = gsum + (size_t)cur * D + lane * VPL;
#pragma unroll
          for (int x = 0; x < VPL; ++x)
            if (!RAGGED || lane * VPL + x < D) o[x] = acc.v[x];
        }
      } else {
        const int h = starts_here ? 1 : 0;
#pragma unroll
        for (int x = 0; x < VPL; ++x) part[w][h][lane * VPL + x] = acc.v[x];
        if (lane == 0) {
          if (h == 0) head_state[w] = ends_here ? 1 : 2;
          else tail_u[w] = cur;
        }
      }
    };
    // The row of a slot.  Its address is a scalar and a lane's offset: formed in vector registers it shared them
    // with loads in flight, and every load waited for the one before (55 -> 74 us at 500,000 Zipf ids).
    auto load_row = [&](int slot, LaneVec<VPL>& r) {
      const float* row = grad + (size_t)(uint32_t)lane_value((int)myb, slot) * D;
      if constexpr (RAGGED) {
#pragma unroll
        for (int x = 0; x < VPL; ++x)  // lanes past the row's end read its last float; nothing stores them
          r.v[x] = __builtin_nontemporal_load(row + (uint32_t)min(lane * VPL + x, D - 1));
      } else {
        stream_load<VPL>(row + (uint32_t)(lane * VPL), r.v);
      }
    };
    auto add_row = [&](int slot, int end, const LaneVec<VPL>& r) {  // end: where the run before it ends
      const int u = lane_value(mysu, slot);
      if (u != cur) {
        flush(end);
        cur = u;
        cur_first = slot;
#pragma unroll
        for (int x = 0; x < VPL; ++x) acc.v[x] = 0.f;
      }
#pragma unroll
      for (int x = 0; x < VPL; ++x) acc.v[x] += r.v[x];
    };
    if (__popcll(need_mask) <= sparse_slots(VPL, RAGGED)) {
      // the slots there are, in order; of a round with fewer the last one is read again and not added
      unsigned long long left = need_mask;
      int end = 0;
      auto round = [&](auto rows) {
        constexpr int ROWS = decltype(rows)::value;
        LaneVec<VPL> r[ROWS];
        unsigned long long ahead = left;
        const int n = min(__popcll(left), ROWS);
#pragma unroll
        for (int k = 0; k < ROWS; ++k) {
          load_row(__ffsll((long long)ahead) - 1, r[k]);
          if (k + 1 < n) ahead &= ahead - 1;
        }
        TT_LOADS_DONE();
#pragma unroll
        for (int k = 0; k < ROWS; ++k)
          if (k < n) {  // uniform
            const int slot = __ffsll((long long)left) - 1;
            left &= left - 1;
            add_row(slot, end, r[k]);
            end = slot + 1;
          }
      };
      while (left) {
        if (VPL > 1 && __popcll(left) > 8) round(std::integral_constant<int, 16>{});
        else round(std::integral_constant<int, 8>{});
      }
      flush(end);
    } else {
      // all slots; those that need no row read one that is read anyway, or, where a row is many loads, none (no
      // run of theirs is stored)
      constexpr bool kSkip = RAGGED && VPL > 1;
      const int spare = __ffsll((long long)need_mask) - 1;
      LaneVec<VPL> r[kRows];
      if constexpr (kSkip) {
#pragma unroll
        for (int k = 0; k < kRows; ++k)
#pragma unroll
          for (int x = 0; x < VPL; ++x) r[k].v[x] = 0.f;
      }
      for (int half = 0; half < kWave / kRows; ++half) {
        if (half * kRows >= nv) break;
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
          const int slot = half * kRows + k;
          const bool on = (need_mask >> slot) & 1ull;
          if (!kSkip || on) load_row(on ? slot : spare, r[k]);
        }
        TT_LOADS_DONE();
#pragma unroll
        for (int k = 0; k < kRows; ++k)
          if (half * kRows + k < nv) add_row(half * kRows + k, half * kRows + k, r[k]);
      }
      flush(nv);
    }
    __syncthreads();
    // join the pieces inside the block, in wave order
    // (a) the run that begins in this wave's tail
    if (tail_u[w] >= 0) {
      LaneVec<VPL> t;
#pragma unroll
      for (int x = 0; x < VPL; ++x) t.v[x] = part[w][1][lane * VPL + x];
      bool open = true;
      for (int k = w + 1; k < kGsumWaves && open; ++k) {
        if (head_state[k] == 0) {  // cannot happen for a run that continues; keeps the loop safe
          open = false;
          break;
        }
#pragma unroll
        for (int x = 0; x < VPL; ++x) t.v[x] += part[k][0][lane * VPL + x];
        if (head_state[k] == 1) open = false;
      }
      if (open && lane == 0) atomicOr(&ctr->err, 16);  // a run left the block: entries never do
      float* o = gsum + (size_t)tail_u[w] * D;
#pragma unroll
      for (int x = 0; x < VPL; ++x)
        if (!RAGGED || lane * VPL + x < D) o[lane * VPL + x] = t.v[x];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// dispatch

bool mfma_shape(const Shape& s) {
  return s.d1 == 4 && s.d2 == 4 && s.r1 == s.r2 &&
         (s.r1 == 8 || s.r1 == 16 || s.r1 == 32 || s.r1 == 64 || s.r1 == 128) &&
         (s.d3 == 4 || s.d3 == 8);
}

static inline int cdivi(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
static inline int grid_cap(int64_t items, int cap) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(items, cap));
}
constexpr int kMGridCap = 256 * 8;

// Blocks of `threads` threads of a kernel that the current device holds at once (what the
// runtime's occupancy calculation says for the kernel's registers and LDS, times the compute
// units).  The per-chunk kernels launch that many blocks at most and walk their work units with
// the grid's stride: every block is resident from the start, none waits for another to end.
template <class K>
static int resident_blocks(K kernel, int threads) {
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
      per_cu < 1)
    per_cu = 8;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  return per_cu * cus;
}

#define TT_DISPATCH_R(R_, CALL)      \
  switch (R_) {                      \
    case 16: { constexpr int R = 16; CALL; } break; \
    case 32: { constexpr int R = 32; CALL; } break; \
    case 64: { constexpr int R = 64; CALL; } break; \
    default: { constexpr int R = 128; CALL; } break; \
  }
// the kernels that also exist for rank 8 (prefix products and rows; rank 8 takes the fused middle
// kernel in the backward pass)
#define TT_DISPATCH_R8(R_, CALL)                    \
  if ((R_) == 8) {                                  \
    constexpr int R = 8;                            \
    CALL;                                           \
  } else {                                          \
    TT_DISPATCH_R(R_, CALL)                         \
  }
// Blocks of a wide kernel: no more than the device holds at once, each walks the units with the
// grid's stride (the bound on the units is known here, their number only on the device: clustered
// ids leave it thirty times smaller, and dispatching blocks that find nothing costs more than the
// work).
template <class K>
static int wide_grid(int* slots, K kernel, int64_t units) {
  if (*slots == 0) *slots = resident_blocks(kernel, kMThreads);
  return grid_cap(units, *slots);
}

void launch_prefix_fwd_mfma(const Plan& pl, const Workspace& ws, const float* g1, const float* g2,
                            int B, hipStream_t st) {
  const int64_t chunks = cdivi(std::min<int64_t>(B, pl.maxQ), kChunk2) + pl.sh.n2;
#define TT_PF(RR)                                                                                  \
  k_prefix_fwd_mfma<RR><<<(int)(chunks * pf_units(RR)), kWave, 0, st>>>(g1, g2, ws.c2_item,        \
                                                                        ws.c2_desc, ws.P, ws.ctr)
#define TT_PW(RR)                                                                                  \
  k_prefix_fwd_wide<RR><<<wide_grid(&pl.unit_slots[0], k_prefix_fwd_wide<RR>, chunks * (4 * RR / 128)), \
                          kMThreads, 0, st>>>(g1, g2, ws.c2_item, ws.c2_desc, ws.P, ws.ctr)
  switch (pl.sh.r1) {
    case 8: TT_PF(8); break;
    case 16: TT_PF(16); break;
    case 32: TT_PF(32); break;
    case 64: TT_PW(64); break;
    default: TT_PW(128); break;
  }
#undef TT_PF
#undef TT_PW
}

void launch_prefix_bwd_mfma(const Plan& pl, const Workspace& ws, const float* g1, const float* g2,
                            int B, hipStream_t st) {
  const int64_t chunks = cdivi(std::min<int64_t>(B, pl.maxQ), kChunk2) + pl.sh.n2;
#define TT_PB(RR)                                                                                  \
  k_prefix_bwd_wide<RR><<<wide_grid(&pl.unit_slots[1], k_prefix_bwd_wide<RR>, chunks * (4 * RR / 128 + 1)), \
                          kMThreads, 0, st>>>(g1, g2, ws.dPsum, ws.c2_item, ws.c2_desc, ws.dg1part, \
                                              ws.part2, ws.ctr)
  if (pl.sh.r1 == 64) TT_PB(64); else TT_PB(128);
#undef TT_PB
}

void launch_id_bwd_mfma(const Plan& pl, const Workspace& ws, const float* g3, const float* grad,
                        int B, hipStream_t st) {
  // both roles loop over their work with a stride of half the grid
  const int64_t waves_q = std::min<int64_t>(B, pl.maxQ), waves_c = cdivi(B, chunk3_fill(B)) + (int64_t)pl.sh.n3;
  const int per_role = kXcds * grid_cap(cdivi(std::max(waves_q, waves_c), kMWaves * kXcds), kMGridCap / kXcds);
#define TT_ID(RR, DD)                                                                              \
  k_id_bwd_mfma<RR, DD><<<2 * per_role, kMThreads, 0, st>>>(g3, ws.P, grad, ws.gsum, ws.u_code,    \
                                                            ws.u_i3, ws.q_us, ws.c3_item,          \
                                                            ws.c3_desc, ws.dPsum, ws.part3, ws.ctr)
  if (pl.sh.r1 == 64) {
    if (pl.sh.d3 == 4) TT_ID(64, 4); else TT_ID(64, 8);
  } else {
    if (pl.sh.d3 == 4) TT_ID(128, 4); else TT_ID(128, 8);
  }
#undef TT_ID
}

// true when k_bwd_mid_mfma covers the shape (else: k_id_bwd_mfma followed by k_prefix_bwd_wide)
bool mfma_fused_mid(const Shape& s) { return mfma_shape(s) && s.r1 <= 32; }

void launch_bwd_mid_mfma(const Plan& pl, const Workspace& ws, const float* g1, const float* g2,
                         const float* g3, const float* grad, int B, hipStream_t st) {
  const int chunk_blocks = cdivi(std::min<int64_t>(B, pl.maxQ), kChunk2) + (int)pl.sh.n2;
  // fewer than four ids per prefix of the table: blocks of four wavefronts (figures at the kernel)
  const bool narrow = pl.sh.r1 <= 16 && B < 4 * (int64_t)pl.sh.n1 * pl.sh.n2;
  const int waves = narrow ? 4 : 8;
  // the same number of by-i3 blocks on every XCD
  const int dg3_blocks =
      kXcds * cdivi(cdivi(cdivi(B, chunk3_fill(B)) + (int64_t)pl.sh.n3, kXcds), waves);
  auto launch = [&](auto kernel) {
    kernel<<<chunk_blocks + dg3_blocks, waves * kWave, 0, st>>>(
        g1, g2, g3, ws.P, grad, ws.gsum, ws.u_code, ws.u_i3, ws.c2_item, ws.c2_desc, ws.c3_item, ws.c3_desc,
        ws.walk3, ws.dg1part, ws.part2, ws.part3, chunk_blocks, ws.ctr);
  };
  if (pl.sh.r1 == 8) {
    if (narrow) pl.sh.d3 == 4 ? launch(k_bwd_mid_mfma<8, 4, 4>) : launch(k_bwd_mid_mfma<8, 8, 4>);
    else pl.sh.d3 == 4 ? launch(k_bwd_mid_mfma<8, 4, 8>) : launch(k_bwd_mid_mfma<8, 8, 8>);
  } else if (pl.sh.r1 == 16) {
    if (narrow) pl.sh.d3 == 4 ? launch(k_bwd_mid_mfma<16, 4, 4>) : launch(k_bwd_mid_mfma<16, 8, 4>);
    else pl.sh.d3 == 4 ? launch(k_bwd_mid_mfma<16, 4, 8>) : launch(k_bwd_mid_mfma<16, 8, 8>);
  } else {
    pl.sh.d3 == 4 ? launch(k_bwd_mid_mfma<32, 4, 8>) : launch(k_bwd_mid_mfma<32, 8, 8>);
  }
}

void launch_row_fwd_mfma(const Plan& pl, const Workspace& ws, const float* g3, int B, bool beside, float* out,
                         hipStream_t st) {
  const int slots = row_slots(pl.sh.r1, pl.sh.d3, beside, B);
  auto launch = [&](auto kernel) {
    kernel<<<cdivi(cdivi(B, slots), kMWaves), kMThreads, 0, st>>>(B, g3, ws.P, ws.s_rec, out, ws.ctr);
  };
#define TT_ROW(D3_)                                                                                  \
  TT_DISPATCH_R8(pl.sh.r1, {                                                                         \
    if constexpr (R <= 32) {                                                                         \
      if (slots == 8) launch(k_row_fwd_mfma<R, D3_, 8>);                                             \
      else if (slots == 16) launch(k_row_fwd_mfma<R, D3_, 16>);                                      \
      else launch(k_row_fwd_mfma<R, D3_, 32>);                                                       \
    } else {                                                                                         \
      launch(k_row_fwd_mfma<R, D3_, 16>);                                                            \
    }                                                                                                \
  })
  if (pl.sh.d3 == 4) {
    TT_ROW(4)
  } else {
    TT_ROW(8)
  }
#undef TT_ROW
}

void launch_gsum_block(const Plan& pl, const Workspace& ws, const float* grad, int B,
                       hipStream_t st) {
  const int grid = grid_cap(cdivi(B, kGsumBlockSlots), kMGridCap);
  const uint32_t* perm = ws.val[pl.keys.sorted()];
  const int D = pl.sh.D;
  auto launch = [&](auto kernel) {
    kernel<<<grid, kGsumThreads, 0, st>>>(B, D, grad, ws.s_u, perm, ws.gsum, ws.ctr);
  };
  if (D == 64) launch(k_gsum_block<1, false>);
  else if (D == 128) launch(k_gsum_block<2, false>);
  else if (D <= 64) launch(k_gsum_block<1, true>);
  else if (D <= 128) launch(k_gsum_block<2, true>);
  else launch(k_gsum_block<4, true>);
}

// rows this long have a block version of the gradient sums (any shape)
bool gsum_block_rows(const Shape& s) { return s.D <= 4 * kWave; }

}  // namespace ttemb
