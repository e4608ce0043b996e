// Any-shape kernels with their products on the matrix cores (gfx950, fp32): prefixes of up to 32 lines
// d1*d2, ranks up to 64, d3 up to 16.  Larger shapes, and forms of these that are slower here (any_*_takes),
// take the kernels of tt_emb_compute.hip.
//
// The products of this path are small and of any size, so every operand goes from memory (or an LDS tile)
// straight to the registers of v_mfma_f32_16x16x4f32, whose lane (kg, l16) = (lane/16, lane%16) holds
// A[i = l16][k = kg], B[k = kg][j = l16] and D[i = 4kg + v][j = l16].  Indices past an edge are clamped to
// one that exists: what they add to rows and columns that do not exist is dropped, and where they would
// lengthen a sum both operands are set to zero (zero times an infinity is not zero).  The loads of a step
// stand in one block in front of its products, so that they are in flight together.  Sizes are known at run
// time only: what these kernels spend is mostly instructions, so whatever does not change is formed once, and
// indices are divided by multiplication.
#include <algorithm>

#include "tt_emb_internal.h"

namespace ttemb {

__device__ __forceinline__ f4 mfma_any(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ const float* grad_row(int code, const float* __restrict__ grad,
                                                 const float* __restrict__ gsum, int D) {
  return code >= 0 ? grad + (size_t)code * D : gsum + (size_t)(-code - 1) * D;
}
__device__ __forceinline__ int lane_of(int v, int src) {
  return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(src));
}
// x / d for 0 <= x < 2^20 / d, with inv = ceil(2^20 / d)
__device__ __forceinline__ int divided(int x, uint32_t inv) { return (int)(((uint32_t)x * inv) >> 20); }
// e / d for 0 <= e < 2^21, with inv = 1 / d: half a unit keeps the product off the integers
__device__ __forceinline__ int quotient(int e, float inv) { return (int)(((float)e + 0.5f) * inv); }
static inline uint32_t inverse_of(int d) { return ((1u << 20) + (uint32_t)d - 1) / (uint32_t)d; }
__host__ __device__ constexpr int up16(int x) { return (x + 15) & ~15; }
__device__ constexpr int up64(int x) { return (x + 63) & ~63; }
template <bool VEC>
struct AnyWord {
  typedef float type;
};
template <>
struct AnyWord<true> {
  typedef f4 type;
};

// ---------------------------------------------------------------------------------------------
// The middle of the backward pass of one by-i2 chunk (<= 16 prefixes), without its dPsum in memory:
//   (i)   dPsum_q = sum over the ids u of q of g_u G3[i3(u)]^T, contraction index (u, j3), one wavefront
//         per prefix: gradient rows and G3 slices of `fill` ids at a time go to LDS as they lie in memory
//         (the next ids' are in flight meanwhile), and the operands are read from there
//   (ii)  dg1part[q] = dPsum_q G2[i2]^T, both operands from LDS
//   (iii) part2 of the chunk = sum over its prefixes of G1[i1]^T dPsum_q
// MT, NT: tiles of 16 that the d1*d2 lines and the r2 columns (and r1 lines) of the products need.
// 200,000 Zipf ids of (125,140,140) x (4,5,5), rank 32: 61 us; as kernels of their own (dPsum through memory,
// operands fetched sixteen deep behind barriers) the steps took 40 + 99.  Where the time goes: 26 us without
// (i) (staging, steps (ii) and (iii), 1200 blocks on two places a compute unit); (i) is bound by the
// instructions around its loads and by the prefix with the most ids in a block.  Operands read element by
// element from memory, whose addresses cost several instructions and a line each, took 92.
constexpr int kAnyWaves = 8;
struct AnyMidLds {  // strides and floats of a block's dynamic LDS
  int ws, as, t, b, a;
  static constexpr int kWords = 24;  // floats of them that a lane has in flight
  int per, fill, room;  // floats of an id's operands; ids of a wavefront in LDS at a time, in the memory of T
  __host__ __device__ explicit AnyMidLds(const Shape& s) {
    ws = up16(s.W) + 4;
    as = up16(s.r1) + 4;
    b = up16(s.r1) * ws;
    a = kChunk2 * s.d1 * as;
    const int tile = kChunk2 * s.d1 * ws;
    per = s.D + s.S3;
    fill = (tile > 8192 ? tile : 8192) / (kAnyWaves * per);
    fill = fill > kWords * kWave / per ? kWords * kWave / per : fill;
    fill = fill < 1 ? 1 : fill > kWave ? kWave : fill;
    if (fill >= 4) fill &= ~3;
    room = per * ((fill + 3) & ~3);
    t = tile > kAnyWaves * room ? tile : kAnyWaves * room;
  }
  __host__ __device__ int floats() const { return t + b + a; }
};

// VEC: rows of gradients and slices of G3 are whole 16-byte words, and aligned
template <int MT, int NT, bool VEC>
__global__ __launch_bounds__(kAnyWaves * kWave, 4) void k_any_mid(
    Shape sh, uint32_t inv_d1, uint32_t inv_d2, const float* __restrict__ g1, const float* __restrict__ g2,
    const float* __restrict__ g3, const float* __restrict__ grad, const float* __restrict__ gsum,
    const int* __restrict__ u_code, const int* __restrict__ u_i3, const int4* __restrict__ c2_item,
    const int4* __restrict__ c2_desc, float* __restrict__ dg1part, float* __restrict__ part2,
    const Counters* __restrict__ ctr) {
  extern __shared__ __align__(16) float lds[];
  constexpr int kT = kAnyWaves * kWave;
  const AnyMidLds at(sh);
  float *T = lds, *Bl = T + at.t, *A1 = Bl + at.b;
  __shared__ int q_of[kChunk2];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave, l16 = lane % 16, kg = lane / 16;
  const int wp = at.ws - 4;
  // descriptor, records and count are read together (the grid never exceeds the tables)
  const int c = blockIdx.x;
  const int4 desc = c2_desc[c], item = c2_item[(size_t)c * kChunk2 + tid % kChunk2];
  if (c >= ctr->nchunk2) return;
  const int cnt = desc.z, rows = cnt * sh.d1, rows16 = up16(rows);
  const float* Bm = g2 + (size_t)desc.x * sh.S2;
  if (tid < kChunk2) q_of[tid] = item.x;  // records past the chunk's count are unwritten
  // this wavefront's prefixes w and w + 8: where the operands of their first 64 ids lie, one id a lane
  typedef typename AnyWord<VEC>::type word;
  constexpr int WD = VEC ? 4 : 1;
  int u0[2], nu[2];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int t = w + g * kAnyWaves;
    u0[g] = lane_of(item.z, t);
    nu[g] = t < cnt ? lane_of(item.w, t) - u0[g] : 0;  // a prefix has an id at least
  }
  struct Operands {
    int lo, hi, slice;  // address of the gradient row, offset of the G3 slice
  };
  auto point = [&](int g, int ub) {
    const int u = u0[g] + ub + min(lane, nu[g] - ub - 1);
    const uintptr_t row = (uintptr_t)grad_row(u_code[u], grad, gsum, sh.D);
    return Operands{(int)(uint32_t)row, (int)(row >> 32), u_i3[u] * sh.S3};
  };
  Operands now{0, 0, 0}, then{0, 0, 0};
  if (nu[0] > 0) now = point(0, 0);
  if (nu[1] > 0) then = point(1, 0);
  // G2[i2], zero from column W to the end of its last tile of 16
  if (sh.W % 4 == 0) {
    const float inv = 4.f / (float)wp;
    for (int e = tid; e < sh.r1 * (wp / 4); e += kT) {
      const int r = quotient(e, inv), col = (e - r * (wp / 4)) * 4;
      f4 v = f4{0.f, 0.f, 0.f, 0.f};
      if (col < sh.W) v = *(const f4*)(Bm + (size_t)r * sh.W + col);
      *(f4*)(Bl + r * at.ws + col) = v;
    }
  } else {
    const float inv = 1.f / (float)wp;
    for (int e = tid; e < sh.r1 * wp; e += kT) {
      const int r = quotient(e, inv), col = e - r * wp;
      Bl[r * at.ws + col] = col < sh.W ? Bm[(size_t)r * sh.W + col] : 0.f;
    }
  }
  // lines of G1, zero past the chunk's (lane t of every wavefront holds record t)
  {
    const float inv = 1.f / (float)sh.r1;
    for (int e = tid; e < up64(rows16 * sh.r1); e += kT) {
      const int r = quotient(e, inv), a = e - r * sh.r1, t = min(divided(r, inv_d1), cnt - 1);
      const float v = g1[(size_t)__shfl(item.y, t) * sh.S1 + min(r - t * sh.d1, sh.d1 - 1) * sh.r1 + a];
      if (r < rows16) A1[r * at.as + a] = r < rows ? v : 0.f;
    }
  }
  // (i)
  f4 acc[2][MT][NT];  // prefix w, then w + 8
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[g][mt][nt] = f4{0.f, 0.f, 0.f, 0.f};
  if (w < cnt) {
    constexpr int kWords = AnyMidLds::kWords / WD;  // words of a lane in flight
    const int nd = sh.D / WD, per_id = at.per / WD;
    const float inv_per = 1.f / (float)per_id;
    float* mine = T + w * at.room;
    int a_at[MT], b_at[NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) a_at[mt] = min(16 * mt + l16, sh.M - 1) * sh.d3;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) b_at[nt] = sh.D + min(16 * nt + l16, sh.r2 - 1) * sh.d3;
    word v[kWords];
    auto fetch = [&](int f0, int n) {  // operands of ids f0 .. of the n that the lanes point at
      const int total = min(at.fill, n - f0) * per_id;
#pragma unroll
      for (int j = 0; j < kWords; ++j) {
        if (j * kWave >= total) break;  // uniform
        const int e = min(lane + j * kWave, total - 1), id = quotient(e, inv_per), x = e - id * per_id;
        const uintptr_t g = (uint32_t)__shfl(now.lo, f0 + id) | (uintptr_t)__shfl(now.hi, f0 + id) << 32;
        const float* s3 = g3 + (uint32_t)__shfl(now.slice, f0 + id);
        const word* from = x < nd ? (const word*)g + x : (const word*)s3 + (x - nd);
        v[j] = *from;
      }
    };
    auto multiply = [&](f4 (&sum)[MT][NT], int here) {
      for (int id0 = 0; id0 < here; id0 += 4) {
        const float* src = mine + (id0 + kg) * at.per;
#pragma unroll 4
        for (int j3 = 0; j3 < sh.d3; ++j3) {
          float a[MT], b[NT];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) a[mt] = src[a_at[mt] + j3];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) b[nt] = src[b_at[nt] + j3];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) sum[mt][nt] = mfma_any(a[mt], b[nt], sum[mt][nt]);
        }
      }
    };
    int g = 0, ub = 0, f0 = 0, n = min(kWave, nu[0]);
    fetch(0, n);
    for (bool more = true; more;) {
      const int here = min(at.fill, n - f0), here4 = (here + 3) & ~3, was = g;
      wave_sync();  // the previous fill has been read
#pragma unroll
      for (int j = 0; j < kWords; ++j) {
        const int e = lane + j * kWave;
        if (e < here * per_id) *(word*)(mine + e * WD) = v[j];
      }
      // ids up to a multiple of four count zero
      for (int e = here * at.per + lane; e < here4 * at.per; e += kWave) mine[e] = 0.f;
      wave_sync();
      // the next fill, in flight while this one is multiplied: of the same ids, of the prefix's next 64,
      // of the other prefix
      f0 += at.fill;
      if (f0 >= n) {
        f0 = 0;
        ub += kWave;
        if (ub < nu[g]) {
          now = point(g, ub);
        } else {
          more = g == 0 && nu[1] > 0;
          g = 1;
          ub = 0;
          now = then;
        }
        n = min(kWave, nu[g] - ub);
      }
      if (more) fetch(f0, n);
      if (was == 0) multiply(acc[0], here);
      else multiply(acc[1], here);
    }
  }
  __syncthreads();  // the operands' memory becomes the tile's
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = 16 * mt + 4 * kg + v, j1 = divided(m, inv_d2);
      float* dst = T + j1 * at.ws + (m - j1 * sh.d2) * sh.r2 + l16;
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          if (w + g * kAnyWaves < cnt && m < sh.M && 16 * nt + l16 < sh.r2)
            dst[(w + g * kAnyWaves) * sh.d1 * at.ws + 16 * nt] = acc[g][mt][nt][v];
    }
  // the tile's columns past W and its lines past the chunk's
  if (wp > sh.W)
    for (int e = tid; e < rows16 * (wp - sh.W); e += kT) {
      const int r = e / (wp - sh.W);
      T[r * at.ws + sh.W + e - r * (wp - sh.W)] = 0.f;
    }
  for (int r = rows + w; r < rows16; r += kAnyWaves)
    for (int e = lane; e < sh.W; e += kWave) T[r * at.ws + e] = 0.f;
  __syncthreads();
  // (ii) tiles of 16 lines x 16 columns of dg1part
  const int ct = (sh.r1 + 15) / 16, wt = (sh.W + 15) / 16;
  for (int unit = w; unit < rows16 / 16 * ct; unit += kAnyWaves) {
    const int rt = unit / ct, a0 = (unit % ct) * 16;
    const float *x = T + (rt * 16 + l16) * at.ws + 4 * kg, *y = Bl + min(a0 + l16, sh.r1 - 1) * at.ws + 4 * kg;
    f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};  // two chains: sums of half the length
#pragma unroll 4
    for (int k = 0; k < wt; ++k) {
      const f4 xv = *(const f4*)(x + 16 * k), yv = *(const f4*)(y + 16 * k);
      acc[0] = mfma_any(xv.x, yv.x, acc[0]);
      acc[1] = mfma_any(xv.y, yv.y, acc[1]);
      acc[0] = mfma_any(xv.z, yv.z, acc[0]);
      acc[1] = mfma_any(xv.w, yv.w, acc[1]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = rt * 16 + 4 * kg + v, t = divided(r, inv_d1);
      if (r < rows && a0 + l16 < sh.r1)
        dg1part[(size_t)q_of[t] * sh.S1 + (r - t * sh.d1) * sh.r1 + a0 + l16] = acc[0][v] + acc[1][v];
    }
  }
  // (iii) 16 columns of part2 at a time, all r1 lines of them
  float* dst = part2 + (size_t)c * sh.S2;
  for (int unit = w; unit < wt; unit += kAnyWaves) {
    const int col = unit * 16 + l16;
    f4 acc[NT];
#pragma unroll
    for (int x = 0; x < NT; ++x) acc[x] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int k = 0; k < rows16; k += 16) {
      float a[4][NT], b[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        b[s] = T[(k + 4 * s + kg) * at.ws + col];
#pragma unroll
        for (int x = 0; x < NT; ++x) a[s][x] = A1[(k + 4 * s + kg) * at.as + min(16 * x + l16, sh.r1 - 1)];
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int x = 0; x < NT; ++x) acc[x] = mfma_any(a[s][x], b[s], acc[x]);
    }
#pragma unroll
    for (int x = 0; x < NT; ++x)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (16 * x + 4 * kg + v < sh.r1 && col < sh.W) dst[(size_t)(16 * x + 4 * kg + v) * sh.W + col] = acc[x][v];
  }
}

// ---------------------------------------------------------------------------------------------
// part3[c] = sum over the unique ids u of by-i3 chunk c of P_q(u)^T g_u (r2 x d3), one wavefront per chunk;
// the contraction runs over the lines of the products, four at a time, five steps of two ids in flight.
// 60 -> 23 us at 200,000 Zipf ids of (125,140,140) x (4,5,5), rank 32 (operands through LDS, products on the
// vector ALUs before); 17 us is what its 139 MB take at the rate of gathers beyond an L2.  Five steps are the 20
// lines of that product; of 4 or 16 lines, or a second round of a few, some are loaded for nothing (figures of
// such shapes at any_dg3_takes).
// VEC: r2 = 16*NT, and a lane's loads along a line of P serve the NT tiles (column NT*l16 + t of tile t).
template <int NT, bool VEC>
__global__ __launch_bounds__(256) void k_any_dg3(
    Shape sh, const float* __restrict__ P, const float* __restrict__ grad, const float* __restrict__ gsum,
    const int2* __restrict__ c3_item, const int4* __restrict__ c3_desc, float* __restrict__ part3,
    const Counters* __restrict__ ctr) {
  typedef float vec __attribute__((ext_vector_type(NT)));
  constexpr int kSteps = 5, kIds = 2;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave, l16 = lane % 16, kg = lane / 16;
  const int c = blockIdx.x * 4 + w;
  // the grid may exceed the tables by a part of a block
  if (c >= ctr->nchunk3) return;
  const int2 item = c3_item[(size_t)c * kChunk3 + lane % kChunk3];
  const int cnt = c3_desc[c].z;
  f4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f4{0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < cnt; i0 += kIds)
    for (int m0 = 0; m0 < sh.M; m0 += 4 * kSteps) {
      float p[kIds][kSteps][NT], g[kIds][kSteps];
#pragma unroll
      for (int x = 0; x < kIds; ++x) {
        // records past the chunk's count are unwritten
        const float* pp = P + (size_t)lane_of(item.y, min(i0 + x, cnt - 1)) * sh.PN;
        const float* gp = grad_row(lane_of(item.x, min(i0 + x, cnt - 1)), grad, gsum, sh.D);
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
          const int m = min(m0 + 4 * s + kg, sh.M - 1);
          g[x][s] = gp[m * sh.d3 + min(l16, sh.d3 - 1)];
          if constexpr (VEC && NT > 1) {
            const vec v = *(const vec*)(pp + m * sh.r2 + NT * l16);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) p[x][s][nt] = v[nt];
          } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) p[x][s][nt] = pp[m * sh.r2 + min(16 * nt + l16, sh.r2 - 1)];
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < kIds; ++x) {
        if (i0 + x >= cnt) break;  // uniform
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
          if (m0 + 4 * s >= sh.M) break;  // uniform
          const bool on = m0 + 4 * s + kg < sh.M;
          const float gv = on ? g[x][s] : 0.f;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma_any(on ? p[x][s][nt] : 0.f, gv, acc[nt]);
        }
      }
    }
  float* dst = part3 + (size_t)c * sh.S3;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 4 * kg + v, r = VEC && NT > 1 ? NT * i + nt : 16 * nt + i;
      if (r < sh.r2 && l16 < sh.d3) dst[r * sh.d3 + l16] = acc[nt][v];
    }
}

// ---------------------------------------------------------------------------------------------
// P_q of a by-i2 chunk: one wavefront per 16 columns of the chunk's product, its G2 strip in registers,
// four tiles of 16 lines (d1 = 4: all sixteen prefixes) in flight together.  KQ = r1/4 rounded up: lane
// group kg takes indices KQ*kg ..  VEC: r1 is a multiple of four, lines of G1 are read by 16-byte words.
template <int KQ, bool VEC>
__global__ __launch_bounds__(kWave) void k_any_prefix(Shape sh, uint32_t inv_d1, int tiles,
                                                      const float* __restrict__ g1, const float* __restrict__ g2,
                                                      const int4* __restrict__ c2_desc,
                                                      const int4* __restrict__ c2_item, float* __restrict__ P,
                                                      const Counters* __restrict__ ctr) {
  constexpr int MT = KQ <= 8 ? 4 : 2;
  const int lane = threadIdx.x, l16 = lane % 16, kg = lane / 16;
  const int c = (int)blockIdx.x / tiles, n0 = ((int)blockIdx.x - c * tiles) * 16;
  // the grid never exceeds the tables: descriptor, records and count are read together
  const int4 desc = c2_desc[c], item = c2_item[(size_t)c * kChunk2 + lane % kChunk2];
  if (c >= ctr->nchunk2) return;
  const int cnt = desc.z, rows = cnt * sh.d1;
  const int col = min(n0 + l16, sh.W - 1);
  const float* Bm = g2 + (size_t)desc.x * sh.S2 + col;
  float b[KQ];
#pragma unroll
  for (int j = 0; j < KQ; ++j) b[j] = Bm[(size_t)min(KQ * kg + j, sh.r1 - 1) * sh.W];
#pragma unroll
  for (int j = 0; j < KQ; ++j) b[j] = KQ * kg + j < sh.r1 ? b[j] : 0.f;
  for (int r0 = 0; r0 < rows; r0 += 16 * MT) {
    float a[MT][KQ];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int r = min(r0 + 16 * mt + l16, rows - 1), t = divided(r, inv_d1);
      const float* line = g1 + (size_t)__shfl(item.y, t) * sh.S1 + (r - t * sh.d1) * sh.r1;
      if constexpr (VEC) {
#pragma unroll
        for (int j = 0; j < KQ / 4; ++j) {
          f4 v = *(const f4*)(line + min(KQ * kg + 4 * j, sh.r1 - 4));
          if (KQ * kg + 4 * j >= sh.r1) v = f4{0.f, 0.f, 0.f, 0.f};
          a[mt][4 * j] = v.x;
          a[mt][4 * j + 1] = v.y;
          a[mt][4 * j + 2] = v.z;
          a[mt][4 * j + 3] = v.w;
        }
      } else {
#pragma unroll
        for (int j = 0; j < KQ; ++j) {
          const float v = line[min(KQ * kg + j, sh.r1 - 1)];
          a[mt][j] = KQ * kg + j < sh.r1 ? v : 0.f;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if (r0 + 16 * mt >= rows) break;  // uniform
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < KQ; ++j) acc = mfma_any(a[mt][j], b[j], acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = r0 + 16 * mt + 4 * kg + v, t = min(divided(r, inv_d1), kChunk2 - 1);
        const int q = __shfl(item.x, t);
        if (r < rows && n0 + l16 < sh.W) P[(size_t)q * sh.PN + (size_t)(r - t * sh.d1) * sh.W + n0 + l16] = acc[v];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Rows: one wavefront per tile of TSL sorted slots.  Up to 16/d3 consecutive distinct ids of one prefix
// make a product (d1*d2 x r2) (r2 x ids*d3).  Its operands come into LDS as they lie in memory, those of
// the next product meanwhile in flight: read by the lanes directly, every 16 bytes of P would be a line of
// their own.  Rows pass through LDS, too, and half a wavefront writes a row to each position of its id.
// MT: tiles of 16 lines of P; KQ = r2/4 rounded up, FULL: exactly; VEC: operands are whole 16-byte words;
// V4: so are rows and out.
constexpr int kAnyRowSlots = 12;  // 8: row kernel 41 us at 200,000 Zipf ids, 56 uniform; 12: 43 and 52; 16: 46, 51; 32: 60, 52
template <int MT, int KQ>
struct AnyRowLds {
  int ps, p, c, e;  // stride of a line of P; floats of P, of the G3 slices, of the rows
  __host__ __device__ explicit AnyRowLds(const Shape& s) {
    ps = s.r2 + 4;
    p = (s.M * ps + 3) & ~3;
    c = (16 * s.r2 + 3) & ~3;
    e = 16 * s.M;
  }
  __host__ __device__ int floats() const { return p + c + e; }
};

template <int MT, int KQ, bool VEC, bool FULL, bool V4>
__global__ __launch_bounds__(256) void k_any_row(Shape sh, int B, uint32_t inv_d3, const float* __restrict__ g3,
                                                 const float* __restrict__ P, const int4* __restrict__ s_rec,
                                                 float* __restrict__ out, Counters* ctr) {
  extern __shared__ __align__(16) float lds[];
  constexpr int TSL = kAnyRowSlots, WD = VEC ? 4 : 1;
  constexpr int NP = (MT * 16 * 4 * KQ / WD + kWave - 1) / kWave, NC = (16 * 4 * KQ / WD + kWave - 1) / kWave;
  typedef typename AnyWord<VEC>::type word;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave, l16 = lane % 16, kg = lane / 16;
  const AnyRowLds<MT, KQ> at(sh);
  float *Pl = lds + w * at.floats(), *Cl = Pl + at.p, *E = Cl + at.c;
  const int upt = 16 / sh.d3;  // ids of a product
  const int ul = min(divided(l16, inv_d3), upt - 1), j3 = min(l16 - ul * sh.d3, sh.d3 - 1);
  const int tile = blockIdx.x * 4 + w;
  if (tile * TSL >= B) return;
  const int s = lane < TSL ? tile * TSL + lane : B;
  const int4 rec = s_rec[min(s, B - 1)];  // {unique-id index, batch position, prefix, i3}
  const uint32_t myb = (uint32_t)rec.y;
  const int mysu = s < B ? rec.x : -2;
  if (s < B && myb >= (uint32_t)B) atomicOr(&ctr->err, 4);
  // slots lo .. hi, whose rows are in LDS at row[slot], to the batch
  auto store_rows = [&](int lo, int hi, int row) {
    if constexpr (V4) {
      // a pair of rows a step; where there are more, four pairs: their look-ups and reads overlap
      const int l32 = lane % 32, nw = sh.D / 4;
      int sl = lo;
      if (hi - lo <= 2) {
        const int slot = min(lo + lane / 32, hi - 1);
        const uint32_t b = (uint32_t)__shfl((int)myb, slot);
        const f4* src = (const f4*)(E + __shfl(row, slot) * sh.D);
        if (b < (uint32_t)B && lo + lane / 32 < hi)
          for (int e = l32; e < nw; e += 32) __builtin_nontemporal_store(src[e], (f4*)(out + (size_t)b * sh.D) + e);
        sl = hi;
      }
      for (; sl < hi; sl += 8) {
        uint32_t b[4];
        const f4* src[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int slot = sl + 2 * k + lane / 32, mine = min(slot, hi - 1);
          b[k] = (uint32_t)__shfl((int)myb, mine);
          src[k] = (const f4*)(E + __shfl(row, mine) * sh.D);
          if (slot >= hi) b[k] = 0xffffffffu;
        }
        for (int e = l32; e < nw; e += 32) {
          f4 v[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = src[k][e];
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (b[k] < (uint32_t)B) __builtin_nontemporal_store(v[k], (f4*)(out + (size_t)b[k] * sh.D) + e);
        }
      }
    } else {
      for (int sl = lo; sl < hi; ++sl) {
        const uint32_t b = (uint32_t)lane_of((int)myb, sl);
        const float* src = E + lane_of(row, sl) * sh.D;
        if (b < (uint32_t)B)
          for (int e = lane; e < sh.D; e += kWave) __builtin_nontemporal_store(src[e], out + (size_t)b * sh.D + e);
      }
    }
  };
  const int nv = __popcll(__ballot(mysu >= 0)), ns = min(TSL, B - tile * TSL);
  if (nv < ns) {  // out-of-range ids, the tail of the sorted order: zero rows
    for (int e = lane; e < sh.D; e += kWave) E[e] = 0.f;
    wave_sync();
    store_rows(nv, ns, 0);
    wave_sync();
  }
  if (nv == 0) return;
  const int u_lo = lane_of(mysu, 0), nu = lane_of(mysu, nv - 1) - u_lo + 1;
  // lane e takes the tile's e-th distinct id: its first slot, prefix and i3
  const int before = __shfl_up(mysu, 1);
  const bool first = lane < nv && (lane == 0 || mysu != before);
  const int rank = lane < nv ? mysu - u_lo : nu - 1;
  const int to = first ? rank : nu + lane - rank - 1;
  const int u_slot = __builtin_amdgcn_ds_permute(to * 4, lane);
  const int myq = __builtin_amdgcn_ds_permute(to * 4, rec.z), myi3 = __builtin_amdgcn_ds_permute(to * 4, rec.w);
  // products: every upt-th id of a run of ids with one prefix starts one
  const int q_before = __shfl_up(myq, 1);
  const unsigned long long runs = __ballot(lane < nu && (lane == 0 || myq != q_before));
  const unsigned long long upto = runs & (lane == 63 ? ~0ull : ((2ull << lane) - 1ull));
  const int run_first = 63 - __clzll((long long)(upto | 1ull));
  const unsigned long long groups = __ballot(lane < nu && (lane - run_first) % upt == 0);
  auto end_of = [&](int st) {  // where the product that starts at id st ends
    const unsigned long long after = groups & ~((2ull << st) - 1ull);
    return after ? __ffsll((long long)after) - 1 : nu;
  };
  // where a lane's words of P go in LDS, which id its words of the slices are of: the same for every product
  const int np = sh.PN / WD, s3w = sh.S3 / WD, line_w = sh.r2 / WD;
  const float inv_line = 1.f / (float)line_w, inv_s3w = 1.f / (float)s3w;
  int p_to[NP], c_id[NC];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int e = lane + k * kWave;
    const int line = quotient(e, inv_line);
    p_to[k] = line * at.ps + (e - line * line_w) * WD;
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) c_id[k] = quotient(lane + k * kWave, inv_s3w);
  word pv[NP], cv[NC];
  auto fetch = [&](int st) {
    const int n = end_of(st) - st;
    const word* pq = (const word*)(P + (size_t)lane_of(myq, st) * sh.PN);
#pragma unroll
    for (int k = 0; k < NP; ++k) pv[k] = pq[min(lane + k * kWave, np - 1)];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int id = min(c_id[k], n - 1), x = min(lane + k * kWave - id * s3w, s3w - 1);
      cv[k] = ((const word*)(g3 + (size_t)__shfl(myi3, st + id) * sh.S3))[x];
    }
  };
  fetch(0);
  for (int st = 0; st < nu;) {
    const int end = end_of(st), n = end - st;
    wave_sync();
#pragma unroll
    for (int k = 0; k < NP; ++k)
      if (lane + k * kWave < np) *(word*)(Pl + p_to[k]) = pv[k];
#pragma unroll
    for (int k = 0; k < NC; ++k)
      if (lane + k * kWave < n * s3w) *(word*)(Cl + (lane + k * kWave) * WD) = cv[k];
    wave_sync();
    if (end < nu) fetch(end);  // in flight while this product is formed and stored
    float b[KQ];
    const float* cp = Cl + min(ul, n - 1) * sh.S3 + j3 + (FULL ? KQ * kg * sh.d3 : 0);
#pragma unroll
    for (int j = 0; j < KQ; ++j) {
      const float v = cp[FULL ? j * sh.d3 : min(KQ * kg + j, sh.r2 - 1) * sh.d3];
      b[j] = FULL || KQ * kg + j < sh.r2 ? v : 0.f;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float* pr = Pl + min(16 * mt + l16, sh.M - 1) * at.ps;
      f4 acc = {0.f, 0.f, 0.f, 0.f};
      if (VEC && KQ % 4 == 0) {  // a line's last word may lie past r2: its padding
#pragma unroll
        for (int j = 0; j < KQ; j += 4) {
          f4 v = *(const f4*)(pr + (FULL ? KQ * kg + j : min(KQ * kg + j, sh.r2)));
          if (!FULL && KQ * kg + j >= sh.r2) v = f4{0.f, 0.f, 0.f, 0.f};
          acc = mfma_any(v.x, b[j], acc);
          acc = mfma_any(v.y, b[j + 1], acc);
          acc = mfma_any(v.z, b[j + 2], acc);
          acc = mfma_any(v.w, b[j + 3], acc);
        }
      } else {
#pragma unroll
        for (int j = 0; j < KQ; ++j) {
          const float v = pr[min(KQ * kg + j, sh.r2 - 1)];
          acc = mfma_any(KQ * kg + j < sh.r2 ? v : 0.f, b[j], acc);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = 16 * mt + 4 * kg + v;
        if (m < sh.M && l16 < n * sh.d3) E[ul * sh.D + m * sh.d3 + j3] = acc[v];
      }
    }
    wave_sync();
    store_rows(lane_of(u_slot, st), end < nu ? lane_of(u_slot, end) : nv, rank - st);
    st = end;
  }
}

// ---------------------------------------------------------------------------------------------
// dispatch

static inline int cdiva(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
constexpr size_t kAnyLds = 96 * 1024;  // most LDS of a block

// Which of these kernels a batch takes; the others are those of tt_emb_compute.hip.  Times of a kernel in us,
// those / these, 60,000 ids: "many" uniform ids of n = 40^3, "few" Zipf ids of 140^3, "fewer" uniform ids of
// (400,400,30), i.e. 37, 3 and 0.4 per prefix of the table.
// A launch holds fewer than 2^32 threads: the grid of one that would hold more wraps without an error.  The
// kernels of tt_emb_compute.hip walk their work with a bounded grid.
static bool launchable(int64_t blocks, int threads) { return blocks * threads < (int64_t)1 << 32; }
static int64_t chunks_most(const Plan& pl, int B) { return cdiva(std::min<int64_t>(B, pl.maxQ), kChunk2) + (int64_t)pl.sh.n2; }

static bool many_ids(const Plan& pl, int B) { return B >= 8 * (int64_t)pl.sh.n1 * pl.sh.n2; }

// Against k_u_bwd and k_prefix_bwd together:
//   d, r             ids of a fill   many       few        fewer
//   (4,5,5), 32      4               55 / 40    95 / 43    314 / 124
//   (4,5,5), 30      4, not words    55 / 65    96 / 52    312 / 149
//   (2,3,12), 24     2               55 / 65    62 / 33    175 / 88
//   (2,3,12), 33     2               91 / 128   87 / 88    246 / 255
//   (2,2,2), 60      12              41 / 27    78 / 38    243 / 108
//   (2,2,2), 63      11, not words   40 / 50    78 / 50    245 / 145
//   (4,5,5), 33      4, not words    72 / 195   118 / 139  377 / 423
// (the last with 96 accumulator registers and as many spilled ones: more than 16 lines and ranks above 32).
bool any_mid_takes(const Plan& pl, int B) {
  const Shape& s = pl.sh;
  if (s.M > 32 || s.r1 > 64 || s.r2 > 64 || s.d1 > 16 || s.d3 > 32 ||
      s.D + s.S3 > AnyMidLds::kWords * kWave || AnyMidLds(s).floats() * sizeof(float) > kAnyLds ||
      !launchable(chunks_most(pl, B), kAnyWaves * kWave))
    return false;
  const bool wide = std::max(s.r1, s.r2) > 32, words = s.D % 4 == 0 && s.S3 % 4 == 0;
  const int fill = AnyMidLds(s).fill;
  if (wide && (s.M > 16 || fill < 3)) return false;
  return !many_ids(pl, B) || (fill >= 3 && (words || !wide));
}
// Better in every form: (4,5,5), rank 32: many 45 / 21, few 28 / 17, fewer 68 / 35; (2,2,2), 4: 15 / 9, 11 / 7,
// 21 / 11; (4,4,4), 48: 46 / 30, 26 / 20, 66 / 45; (3,7,3), 63: 76 / 45, 39 / 30, 122 / 87.
bool any_dg3_takes(const Plan& pl, int B) {
  const Shape& s = pl.sh;
  return s.r2 <= 64 && s.d3 <= 16 && s.M <= 64 && launchable(cdiva(cdiva(B, chunk3_fill(B)) + (int64_t)s.n3, 4), 256);
}
// Ranks that are no multiple of four read lines of G1 element by element.  Few / fewer ids, those, these:
//   (4,5,5): rank 15 17 / 41, 14 / 31;  24 21 / 55, 18 / 45;  30 27 / 77, 27 / 84;  33 32 / 97, 47 / 165;
//            40 39 / 124, 28 / 91;  64 56 / 187, 47 / 182
//   (4,4,4): rank 15 13 / 25, 13 / 25;  28 21 / 54, 17 / 42;  30 21 / 56, 23 / 66;  48 32 / 96, 26 / 85
bool any_prefix_takes(const Plan& pl, int B) {
  const Shape& s = pl.sh;
  return s.d1 <= 16 && (s.r1 <= 16 || (s.r1 <= 64 && s.r1 % 4 == 0)) &&
         launchable(chunks_most(pl, B) * cdiva(s.W, 16), kWave);
}
// A wavefront stages a product for few rows, or many:
//   d, r           many       few        fewer
//   (4,5,5), 32    34 / 21    29 / 25    45 / 42
//   (4,5,5), 6     24 / 21    22 / 27    29 / 41
//   (4,5,5), 30    47 / 36    39 / 51    70 / 78
//   (4,5,5), 48    38 / 33    32 / 47    51 / 69
//   (4,5,5), 33    51 / 96    41 / 154   78 / 238
//   (4,4,4), 48    31 / 21    26 / 33    41 / 50
//   (2,2,2), 6     18 / 12    18 / 20    23 / 25
bool any_row_takes(const Plan& pl, int B) {
  const Shape& s = pl.sh;
  if (s.M > 32 || s.r2 > 64 || s.d3 > 16 || !launchable(cdiva(B, 4 * kAnyRowSlots), 256)) return false;
  if (s.r2 <= 4 || (s.r2 <= 32 && s.r2 % 4 == 0)) return true;
  return many_ids(pl, B) && (s.r2 <= 32 || s.r2 % 4 == 0);
}

void launch_any_mid(const Plan& pl, const Workspace& ws, const float* g1, const float* g2, const float* g3,
                    const float* grad, int B, hipStream_t st) {
  const Shape& s = pl.sh;
  const int grid = (int)chunks_most(pl, B);
  const size_t lds = AnyMidLds(s).floats() * sizeof(float);
  auto launch = [&](auto kernel) {
    kernel<<<grid, kAnyWaves * kWave, lds, st>>>(s, inverse_of(s.d1), inverse_of(s.d2), g1, g2, g3, grad, ws.gsum,
                                                 ws.u_code, ws.u_i3, ws.c2_item, ws.c2_desc, ws.dg1part, ws.part2,
                                                 ws.ctr);
  };
  const int r = std::max(s.r1, s.r2), nt = r <= 16 ? 1 : r <= 32 ? 2 : 4;
  const bool vec = s.D % 4 == 0 && s.S3 % 4 == 0 && ((uintptr_t)grad & 15u) == 0;
#define TT_ANY_MID(M_, N_) vec ? launch(k_any_mid<M_, N_, true>) : launch(k_any_mid<M_, N_, false>)
  if (s.M <= 16) {
    if (nt == 1) TT_ANY_MID(1, 1);
    else if (nt == 2) TT_ANY_MID(1, 2);
    else TT_ANY_MID(1, 4);
  } else {
    if (nt == 1) TT_ANY_MID(2, 1);
    else TT_ANY_MID(2, 2);
  }
#undef TT_ANY_MID
}

void launch_any_dg3(const Plan& pl, const Workspace& ws, const float* grad, int B, hipStream_t st) {
  const Shape& s = pl.sh;
  const int grid = cdiva(cdiva(B, chunk3_fill(B)) + (int64_t)s.n3, 4);
  auto launch = [&](auto kernel) {
    kernel<<<grid, 256, 0, st>>>(s, ws.P, grad, ws.gsum, ws.c3_item, ws.c3_desc, ws.part3, ws.ctr);
  };
  if (s.r2 <= 16) launch(k_any_dg3<1, false>);
  else if (s.r2 == 32) launch(k_any_dg3<2, true>);
  else if (s.r2 < 32) launch(k_any_dg3<2, false>);
  else if (s.r2 == 64) launch(k_any_dg3<4, true>);
  else launch(k_any_dg3<4, false>);
}

void launch_any_prefix(const Plan& pl, const Workspace& ws, const float* g1, const float* g2, int B, hipStream_t st) {
  const Shape& s = pl.sh;
  const int chunks = (int)chunks_most(pl, B), tiles = cdiva(s.W, 16);
  auto launch = [&](auto kernel) {
    kernel<<<chunks * tiles, kWave, 0, st>>>(s, inverse_of(s.d1), tiles, g1, g2, ws.c2_desc, ws.c2_item, ws.P, ws.ctr);
  };
  if (s.r1 <= 4) launch(k_any_prefix<1, false>);
  else if (s.r1 <= 16) s.r1 % 4 == 0 ? launch(k_any_prefix<4, true>) : launch(k_any_prefix<4, false>);
  else if (s.r1 <= 32) launch(k_any_prefix<8, true>);
  else if (s.r1 <= 48) launch(k_any_prefix<12, true>);
  else launch(k_any_prefix<16, true>);
}

template <int MT, int KQ>
static void any_row(const Plan& pl, const Workspace& ws, const float* g3, int B, float* out, hipStream_t st) {
  const Shape& s = pl.sh;
  const bool vec = s.r2 % 4 == 0;
  const bool v4 = s.D % 4 == 0 && ((uintptr_t)out & 15u) == 0;
  const size_t lds = (size_t)4 * AnyRowLds<MT, KQ>(s).floats() * sizeof(float);
  auto launch = [&](auto kernel) {
    kernel<<<cdiva(B, 4 * kAnyRowSlots), 256, lds, st>>>(s, B, inverse_of(s.d3), g3, ws.P, ws.s_rec, out, ws.ctr);
  };
  if (s.r2 == 4 * KQ) v4 ? launch(k_any_row<MT, KQ, true, true, true>) : launch(k_any_row<MT, KQ, true, true, false>);
  else if (vec) v4 ? launch(k_any_row<MT, KQ, true, false, true>) : launch(k_any_row<MT, KQ, true, false, false>);
  else v4 ? launch(k_any_row<MT, KQ, false, false, true>) : launch(k_any_row<MT, KQ, false, false, false>);
}

void launch_any_row(const Plan& pl, const Workspace& ws, const float* g3, int B, float* out, hipStream_t st) {
  const Shape& s = pl.sh;
  auto by_lines = [&](auto one, auto two) { (s.M <= 16 ? one : two)(pl, ws, g3, B, out, st); };
  if (s.r2 <= 4) by_lines(any_row<1, 1>, any_row<2, 1>);
  else if (s.r2 <= 16) by_lines(any_row<1, 4>, any_row<2, 4>);
  else if (s.r2 <= 32) by_lines(any_row<1, 8>, any_row<2, 8>);
  else by_lines(any_row<1, 16>, any_row<2, 16>);
}

}  // namespace ttemb
