// Learned hierarchy terminator: a linear convolution closure that predicts
// the truncated level W^(N+1) from W^(N) and replaces Eq. (GMFP) at n = N
// (two states).  The closure is a three-layer 5x5 convolution network over
// (q, p) without biases or activations (the hierarchy is linear, so is the
// closure); its input channels are the four packed components of W^(N) and
// the same four multiplied by p (the analytic terminator (zeta p + c0 d/dp)
// W^(N) is one such map).  The three layers compose exactly into one 13x13
// kernel, which is what the propagation applies.
//
//  - closure_apply_kernel: inference, BF16 inputs and weights on MFMA
//    (v_mfma_f32_16x16x16_bf16), FP32 accumulation;
//  - closure_stats_kernel: FP64 second-moment statistics of training pairs
//    (level n, level n + 1) of a propagated hierarchy;
//  - kernel-stack convolutions / correlations and Adam: gradient descent on
//    the three layers against the quadratic loss the statistics define.
#include <cstdint>

#include "device_common.hpp"
#include "qhfpe_internal.hpp"

namespace qhfpe {

namespace {

typedef short bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// FP32 -> BF16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ unsigned short to_bf16(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// ---------------------------------------------------------------------------
// Inference
// ---------------------------------------------------------------------------
// One task: 4 output q rows of one member over all p.  The 16 input rows
// (q0 - 6 .. q0 + 9) are staged in LDS as BF16, channel-last [row][p][8].
// MFMA tile: M = 16 consecutive p, N = 16 = 4 output rows x 4 components,
// K = 16 taps (dp, ci) of one input row: 13 dp x 8 ci = 104 taps in 7
// chunks per row, 16 rows.  The weights, already in this B layout
// [row][chunk][n][k] (closure_weights_kernel), are held in registers, each
// wave holding those of half the input rows.
constexpr int kRowsOut = 4;
constexpr int kRowsIn = kRowsOut + 2 * kClosureHalf;   // 16
constexpr int kChunks = 7;
constexpr int kTaps = (2 * kClosureHalf + 1) * kClosureIn;  // 104 per input row
// Eight waves: wave w takes the tile pairs w % 4 (+ 4 k) over the input rows
// (w / 4) * 8 .. + 7, holding those rows' weights in registers; the two
// halves of each sum meet in LDS.
constexpr int kApplyWaves = 8;
constexpr int kRowHalves = 2;
constexpr int kRowsPerWave = kRowsIn / kRowHalves;  // 8
constexpr int kTilesAtOnce = 2;  // tiles per wave at once
constexpr int kChains = 2;       // accumulators per tile (even and odd input rows): 4 independent MFMA chains
constexpr int kApplyThreads = 64 * kApplyWaves;

// The channels of one grid point as 8 BF16 values (16 bytes).
template <typename T>
__device__ __forceinline__ uint4 pack_channels(const float c[4], float pa) {
  unsigned short h[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    h[k] = to_bf16(c[k]);
    h[4 + k] = to_bf16(pa * c[k]);
  }
  uint4 w4;
  w4.x = (unsigned)h[0] | ((unsigned)h[1] << 16);
  w4.y = (unsigned)h[2] | ((unsigned)h[3] << 16);
  w4.z = (unsigned)h[4] | ((unsigned)h[5] << 16);
  w4.w = (unsigned)h[6] | ((unsigned)h[7] << 16);
  return w4;
}

// Each workgroup walks a contiguous range of tasks in (member, q group)
// order.  The 16 input rows live in a ring of LDS row slots (row q in slot
// (q + 6) mod 16): the next group of the same member needs 4 new rows only,
// which are loaded into registers while the current group runs on the
// matrix cores, and written to the slots the current group no longer reads.
template <typename T, int NP>
__global__ void __launch_bounds__(kApplyThreads, 1)
    closure_apply_kernel(const T* __restrict__ v, int level, long long member_stride, long long level_stride,
                         long long comp_stride, int nq, int batch, double p0, double dp,
                         const unsigned short* __restrict__ wb, T* __restrict__ out, long long out_stride) {
  __shared__ __align__(16) unsigned short sx[kRowsIn * NP * kClosureIn];
  __shared__ f32x4_t sred[kApplyWaves / kRowHalves][kTilesAtOnce][64];  // second-half partial sums
  constexpr int kNewPer = kRowsOut * NP / kApplyThreads;  // new-row points per thread (1 or 2)
  static_assert(kRowsOut * NP % kApplyThreads == 0, "new rows split evenly over the threads");
  const int tid = threadIdx.x;
  const int groups = (nq + kRowsOut - 1) / kRowsOut;
  const long long ntasks = (long long)groups * batch;
  const long long per = (ntasks + gridDim.x - 1) / gridDim.x;
  const long long t_begin = (long long)blockIdx.x * per;
  const long long t_end = t_begin + per < ntasks ? t_begin + per : ntasks;
  const int lane = tid & 63, wid = tid >> 6;
  const int quad = lane >> 4, li = lane & 15;
  // the B fragments of this wave's input rows stay in its registers: they
  // are the same for every tile and task
  const int tg = wid % (kApplyWaves / kRowHalves), half = wid / (kApplyWaves / kRowHalves);
  bf16x4_t bw[kRowsPerWave][kChunks];
#pragma unroll
  for (int rr = 0; rr < kRowsPerWave; ++rr)
#pragma unroll
    for (int ch = 0; ch < kChunks; ++ch) {
      const int row = half * kRowsPerWave + rr;
      bw[rr][ch] = *reinterpret_cast<const bf16x4_t*>(wb + (((row * kChunks + ch) * 16 + li) * 16 + 4 * quad));
    }
  auto load_point = [&](const T* vb, int q, int a, float c[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = 0.f;
    if (q >= 0 && q < nq) {
#pragma unroll
      for (int k = 0; k < 4; ++k) c[k] = (float)vb[k * comp_stride + (long long)q * NP + a];
    }
  };
  auto slot = [](int q) { return (q + kClosureHalf + kRowsIn) % kRowsIn; };
  float nxt[kNewPer][4];  // the next group's new rows, in flight during the MFMA phase
  bool have_next = false;
  for (long long task = t_begin; task < t_end; ++task) {
    const int b = (int)(task / groups), g = (int)(task % groups);
    const int q0 = g * kRowsOut;
    const T* vb = v + (long long)b * member_stride + (long long)level * level_stride;
    __syncthreads();  // the previous group's MFMA reads of sx are done
    if (!have_next) {
      // first group of a member in this range: all 16 rows
      for (int e = tid; e < kRowsIn * NP; e += kApplyThreads) {
        const int r = e / NP, a = e % NP;
        const int q = q0 - kClosureHalf + r;
        float c[4];
        load_point(vb, q, a, c);
        reinterpret_cast<uint4*>(sx)[slot(q) * NP + a] = pack_channels<T>(c, (float)(p0 + a * dp));
      }
    } else {
      // rows q0 + 6 .. q0 + 9 arrived during the previous group
#pragma unroll
      for (int j = 0; j < kNewPer; ++j) {
        const int e = tid + j * kApplyThreads;
        const int r = e / NP, a = e % NP;
        const int q = q0 + kClosureHalf + r;
        reinterpret_cast<uint4*>(sx)[slot(q) * NP + a] = pack_channels<T>(nxt[j], (float)(p0 + a * dp));
      }
    }
    __syncthreads();
    // the next group's new rows, if it is the same member's
    have_next = task + 1 < t_end && g + 1 < groups;
    if (have_next) {
#pragma unroll
      for (int j = 0; j < kNewPer; ++j) {
        const int e = tid + j * kApplyThreads;
        const int r = e / NP, a = e % NP;
        load_point(vb, q0 + kRowsOut + kClosureHalf + r, a, nxt[j]);
      }
    }
    constexpr int kGroups = kApplyWaves / kRowHalves;
    for (int t0 = tg * kTilesAtOnce; t0 < NP / 16; t0 += kGroups * kTilesAtOnce) {
      f32x4_t acc[kTilesAtOnce][kChains];
#pragma unroll
      for (int u = 0; u < kTilesAtOnce; ++u)
#pragma unroll
        for (int c = 0; c < kChains; ++c) acc[u][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int rr = 0; rr < kRowsPerWave; ++rr) {
        const int row = half * kRowsPerWave + rr;
        const unsigned short* xr = sx + slot(q0 - kClosureHalf + row) * NP * kClosureIn;
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
          // A: lane holds taps k = 4 quad .. 4 quad + 3 of output p = 16 tile + li
          const int kk = ch * 16 + 4 * quad;
#pragma unroll
          for (int u = 0; u < kTilesAtOnce; ++u) {
            bf16x4_t av = {0, 0, 0, 0};
            if (kk < kTaps) {
              const int dpo = kk / kClosureIn, ci0 = kk % kClosureIn;
              const int pin = (16 * (t0 + u) + li + dpo - kClosureHalf + NP) % NP;
              av = *reinterpret_cast<const bf16x4_t*>(xr + pin * kClosureIn + ci0);
            }
            // B (registers): taps k = 4 quad .. 4 quad + 3 of output n = li
            acc[u][rr % kChains] =
                __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bw[rr][ch], acc[u][rr % kChains], 0, 0, 0);
          }
        }
      }
      // the second row half hands its partial sums to the first
      if (half == 1) {
#pragma unroll
        for (int u = 0; u < kTilesAtOnce; ++u) sred[tg][u][lane] = acc[u][0] + acc[u][1];
      }
      __syncthreads();
      if (half == 0) {
        // D: lane holds rows i = 4 quad .. 4 quad + 3 (p) of column n = li
        const int r = li >> 2, co = li & 3;
        const int q = q0 + r;
        if (q < nq) {
#pragma unroll
          for (int u = 0; u < kTilesAtOnce; ++u) {
            const f32x4_t sum = acc[u][0] + acc[u][1] + sred[tg][u][lane];
            T* o = out + (long long)b * out_stride + co * comp_stride + (long long)q * NP + 16 * (t0 + u) + 4 * quad;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = (T)sum[j];
          }
        }
      }
      __syncthreads();  // sred is free again
    }
  }
}

// The 13x13 closure kernel K[dq][dp][ci][co] (FP32) in the B layout of
// closure_apply_kernel: wb[row][chunk][n][k] = K[row - n/4][kk/8][kk%8][n%4]
// with kk = 16 chunk + k, zero outside the kernel.
__global__ void closure_weights_kernel(const float* __restrict__ K, unsigned short* __restrict__ wb) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= kClosureWeightElems) return;
  const int k = e % 16, n = (e / 16) % 16, ch = (e / 256) % kChunks, row = e / (256 * kChunks);
  const int kk = ch * 16 + k;
  const int r = n >> 2, co = n & 3, dq = row - r;
  float w = 0.f;
  if (kk < kTaps && dq >= 0 && dq <= 2 * kClosureHalf) {
    const int dpo = kk / kClosureIn, ci = kk % kClosureIn;
    w = K[((dq * (2 * kClosureHalf + 1) + dpo) * kClosureIn + ci) * kClosureOut + co];
  }
  wb[e] = to_bf16(w);
}

// ---------------------------------------------------------------------------
// Training statistics (FP64)
// ---------------------------------------------------------------------------
// A and C are contractions over the grid points of all members, computed with
// v_mfma_f64_16x16x4 (FP64 inputs and sums).  One product takes four
// consecutive p nodes (K) of a row q:
//   A: rows (ci, s), s = 0, 1: X_ci(q, a - s);  columns (cj, t), t = 0, 1:
//      X_cj(q + D + t, a + e - 12), e even: offsets dq = 12 + D + t, dp = e + s.
//      Only D >= 0 is computed: A[dq][dp][ci][cj] = A[24 - dq][24 - dp][cj][ci].
//   C: rows (ci, s): X_ci(q, a + s - 6);  columns (co, t), t = 0..3:
//      Y_co(q + 6 - D - t, a - e): offsets dq = D + t, dp = e + s.
// A part holds the sums of every e for one D (A: D = 0, 2, .., 12, thirteen e;
// C: D = 0, 4, 8, 12, seven e) in its waves' accumulators.  The operands of
// consecutive e and a overlap (position a + e), so four nodes need one new A
// operand and two new B operands for 13 (7) products; they come from the
// caches directly, one element per lane.
// The rows of all members are split into chunks; a workgroup sums one part
// over one chunk (its waves meet in LDS) and writes a partial, and
// closure_stats_sum_kernel adds the chunks in order: no atomics, a repeated
// call gives the same bits.  Bound by the FP64 matrix rate: 32 members of
// 128 x 128 (32 GFLOP of products, 0.44 ms at the rate of a large FP64 matrix
// product) take 0.73 ms; with one thread per output and vector FMAs they
// took 23.6 ms.
constexpr int kStatWaves = 4;
constexpr int kStatThreads = 64 * kStatWaves;
constexpr int kStatPartsA = kClosureHalf + 1, kStatPartsC = 4;
constexpr int kStatEA = 2 * kClosureHalf + 1, kStatEC = kClosureHalf + 1;
constexpr int kStatParts = kStatPartsA + kStatPartsC + 1;  // + yy

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Offset of a part's values in a chunk's partial (256 per product, row-major
// [16][16]); the last part is the one value of yy.
__host__ __device__ constexpr int stat_part_offset(int part) {
  return part <= kStatPartsA ? part * kStatEA * 256
                             : kStatPartsA * kStatEA * 256 + (part - kStatPartsA) * kStatEC * 256;
}
constexpr int kStatPartial = stat_part_offset(kStatParts - 1) + 1;

// Sums of one part over the rows r0 + wave, r0 + wave + kStatWaves, .. < r1
// (a row: one q of one member).  NE products; STEP: +1 when the B operand
// moves with e (A), -1 when against it (C).
template <typename T, int NP, int NE, int STEP>
__device__ __forceinline__ void stat_rows(const T* v, long long member_stride, long long level_stride,
                                          long long comp_stride, int level, int nq, double p0, double dp, int D,
                                          int r0, int r1, int wid, int lane, f64x4_t (&acc)[NE]) {
  constexpr bool kA = STEP > 0;
  const int i = lane & 15, k = lane >> 4;
  const int ci = i & 7, s = i >> 3;           // row of the A operand
  const int cj = kA ? (i & 7) : (i & 3);      // column of the B operand
  const int t = kA ? (i >> 3) : (i >> 2);
  const int pa = kA ? k - s : k + s - kClosureHalf;  // A: p position relative to the chunk's node
  const int pb = kA ? k - 2 * kClosureHalf : k;      // B: the same at e = 0
  const unsigned bytes = (unsigned)(4 * comp_stride * sizeof(T));
  constexpr unsigned kOut = 0x7fffff00u;             // past every level: reads as zero
  for (int r = r0 + wid; r < r1; r += kStatWaves) {
    const int b = r / nq, q = r % nq;
    const T* lv = v + b * member_stride + level * level_stride;
    const rsrc_t rx = make_rsrc(lv, bytes);
    const rsrc_t ry = make_rsrc(kA ? lv : lv + level_stride, bytes);
    const int qb = kA ? q + D + t : q + kClosureHalf - D - t;
    if (kA && q + D >= nq) continue;
    const bool in = qb >= 0 && qb < nq;
    const unsigned oa = (unsigned)((ci & 3) * comp_stride + (long long)q * NP);
    const unsigned ob = (unsigned)((cj & 3) * comp_stride + (long long)qb * NP);
    auto load_a = [&](int a) { return buf_load<T>(rx, (oa + ((a + pa) & (NP - 1))) * (unsigned)sizeof(T), 0); };
    auto load_b = [&](int a) {
      return buf_load<T>(ry, in ? (ob + ((a + pb) & (NP - 1))) * (unsigned)sizeof(T) : kOut, 0);
    };
    // channels 4..7 are p times channels 0..3
    auto chan_a = [&](T x, int a) {
      const double w = p0 + ((a + pa) & (NP - 1)) * dp;
      return ci < 4 ? (double)x : w * (double)x;
    };
    auto chan_b = [&](T x, int a) {
      const double w = p0 + ((a + pb) & (NP - 1)) * dp;
      return (!kA || cj < 4) ? (double)x : w * (double)x;
    };
    // bv[j]: the B operand of e = 2 j at the current node a
    constexpr int j0 = kA ? NE - 2 : 0, j1 = j0 + 1;  // the operands that a step of four nodes brings in
    double bv[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) bv[j] = chan_b(load_b(STEP * 2 * j), STEP * 2 * j);
    T an = load_a(0);
    // (unrolled twice: unrolled over the whole row, with the operands in a
    // ring instead of shifted, the products took 12% longer)
#pragma unroll 2
    for (int a = 0; a < NP; a += 4) {
      const double av = chan_a(an, a);
      // the next node's operands, in flight during the products (the last
      // node's wrap around and are not used)
      const int e0 = a + 4 + STEP * 2 * j0, e1 = a + 4 + STEP * 2 * j1;
      an = load_a(a + 4);
      const T n0 = load_b(e0), n1 = load_b(e1);
#pragma unroll
      for (int j = 0; j < NE; ++j) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[j], acc[j], 0, 0, 0);
      const double c0 = chan_b(n0, e0), c1 = chan_b(n1, e1);
      if constexpr (kA) {
#pragma unroll
        for (int j = 0; j + 2 < NE; ++j) bv[j] = bv[j + 2];
      } else {
#pragma unroll
        for (int j = NE - 1; j >= 2; --j) bv[j] = bv[j - 2];
      }
      bv[j0] = c0;
      bv[j1] = c1;
    }
  }
}

// the waves' accumulators summed into out[NE][16][16]
template <int NE>
__device__ __forceinline__ void stat_store(f64x4_t (&acc)[NE], double* sh, int wid, int lane, double* out) {
  for (int w = 0; w < kStatWaves; ++w) {
    if (wid == w) {
#pragma unroll
      for (int j = 0; j < NE; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // D layout of the FP64 product: row 4 r + lane / 16, column lane % 16
          double* d = sh + j * 256 + (4 * r + (lane >> 4)) * 16 + (lane & 15);
          *d = w == 0 ? acc[j][r] : *d + acc[j][r];
        }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < NE * 256; e += kStatThreads) out[e] = sh[e];
}

// grid (kStatParts, chunks); partial: chunks x kStatPartial doubles
template <typename T, int NP>
__global__ void __launch_bounds__(kStatThreads, 2)
    closure_stats_kernel(const T* __restrict__ v, int level, long long member_stride, long long level_stride,
                         long long comp_stride, int nq, int batch, double p0, double dp, int rows_per_chunk,
                         double* __restrict__ partial) {
  __shared__ double sh[kStatEA * 256];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = blockIdx.x, rows = nq * batch;
  const int r0 = blockIdx.y * rows_per_chunk, r1 = min(rows, r0 + rows_per_chunk);
  double* const out = partial + (long long)blockIdx.y * kStatPartial + stat_part_offset(part);
  if (part < kStatPartsA) {
    f64x4_t acc[kStatEA];
#pragma unroll
    for (int j = 0; j < kStatEA; ++j) acc[j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    stat_rows<T, NP, kStatEA, 1>(v, member_stride, level_stride, comp_stride, level, nq, p0, dp, 2 * part, r0, r1,
                                 wid, lane, acc);
    stat_store<kStatEA>(acc, sh, wid, lane, out);
  } else if (part < kStatPartsA + kStatPartsC) {
    f64x4_t acc[kStatEC];
#pragma unroll
    for (int j = 0; j < kStatEC; ++j) acc[j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    stat_rows<T, NP, kStatEC, -1>(v, member_stride, level_stride, comp_stride, level, nq, p0, dp,
                                  4 * (part - kStatPartsA), r0, r1, wid, lane, acc);
    stat_store<kStatEC>(acc, sh, wid, lane, out);
  } else {
    double acc = 0.0;
    for (int r = r0 + wid; r < r1; r += kStatWaves) {
      const T* ly = v + (r / nq) * member_stride + (level + 1) * level_stride + (long long)(r % nq) * NP;
#pragma unroll
      for (int c = 0; c < kClosureOut; ++c)
#pragma unroll
        for (int a = 0; a < NP; a += 64) {
          const double y = (double)ly[c * comp_stride + a + lane];
          acc = fma(y, y, acc);
        }
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) sh[wid] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0.0;
      for (int w = 0; w < kStatWaves; ++w) s += sh[w];
      *out = s;
    }
  }
}

// stats += the chunks' partials: four threads per output, a quarter of the
// chunks each
constexpr int kSumOutputs = 64;
__global__ void __launch_bounds__(4 * kSumOutputs)
    closure_stats_sum_kernel(const double* __restrict__ partial, int chunks, double* __restrict__ stats) {
  __shared__ double sh[4][kSumOutputs];
  constexpr int H2 = 2 * kClosureHalf, NA = 2 * H2 + 1, NCK = 2 * kClosureHalf + 1;
  const int quarter = threadIdx.x / kSumOutputs;
  const int out = blockIdx.x * kSumOutputs + threadIdx.x % kSumOutputs;
  const int e = min(out, kClosureStatsSize - 1);
  int at;
  if (e < kClosureStatsA) {
    int cj = e % kClosureIn, ci = (e / kClosureIn) % kClosureIn;
    int dpo = e / (kClosureIn * kClosureIn) % NA, dq = e / (kClosureIn * kClosureIn * NA);
    if (dq < H2) {
      dq = 2 * H2 - dq;
      dpo = 2 * H2 - dpo;
      const int c = ci;
      ci = cj;
      cj = c;
    }
    const int D = dq - H2;
    at = stat_part_offset(D / 2) + (dpo / 2) * 256 + ((dpo & 1) * 8 + ci) * 16 + (D & 1) * 8 + cj;
  } else if (e < kClosureStatsA + kClosureStatsC) {
    const int f = e - kClosureStatsA;
    const int co = f % kClosureOut, ci = (f / kClosureOut) % kClosureIn;
    const int dpo = f / (kClosureIn * kClosureOut) % NCK, dq = f / (kClosureIn * kClosureOut * NCK);
    at = stat_part_offset(kStatPartsA + dq / 4) + (dpo / 2) * 256 + ((dpo & 1) * 8 + ci) * 16 + (dq & 3) * 4 + co;
  } else {
    at = stat_part_offset(kStatParts - 1);
  }
  double s = 0.0;
#pragma unroll 8
  for (int c = quarter; c < chunks; c += 4) s += partial[(long long)c * kStatPartial + at];
  sh[quarter][threadIdx.x % kSumOutputs] = s;
  __syncthreads();
  if (quarter == 0 && out < kClosureStatsSize)
    stats[e] += (s + sh[1][threadIdx.x]) + (sh[2][threadIdx.x] + sh[3][threadIdx.x]);
}

// ---------------------------------------------------------------------------
// Training: kernel stacks P[i][a][b] with a 2-D tap index i over an s x s
// square (offsets centred), composed and differentiated exactly: FP32 stacks,
// products and sums in FP64.  The work of an iteration is small (29 million
// multiply-adds); what counts is that no output is one long chain of loads.
// Every sum is therefore split over lanes (or over the waves of a workgroup)
// and its taps are unrolled, so that a lane has a whole row of taps in
// flight, and the five dependent phases of an iteration are five launches:
// W12, K, gradient of K, (G3 + its Adam update | G12), (G1 | G2 and their
// updates).  An iteration takes 40 us (five launches of 7 to 11 us, each a
// round of loads and a reduction long); as eight launches with one thread
// per output it took 440 us.
// ---------------------------------------------------------------------------
constexpr int kStackThreads = 256;

// four consecutive floats, aligned as floats (callers' kernels and states
// need not be aligned to 16 bytes); one 16-byte access
struct Four {
  float x, y, z, w;
};

__device__ __forceinline__ double dot4(Four p, Four q, double acc) {
  acc = fma((double)p.x, (double)q.x, acc);
  acc = fma((double)p.y, (double)q.y, acc);
  acc = fma((double)p.z, (double)q.z, acc);
  return fma((double)p.w, (double)q.w, acc);
}

// One parameter's Adam step: w <- w - lr mhat / (sqrt(vhat) + eps).
struct Adam {
  float lr, b1, b2, c1, c2, eps;
  float* m;
  float* v;
};
__device__ __forceinline__ float adam_step(const Adam& o, int e, float w, float g) {
  const float mi = o.b1 * o.m[e] + (1.f - o.b1) * g;
  const float si = o.b2 * o.v[e] + (1.f - o.b2) * g * g;
  o.m[e] = mi;
  o.v[e] = si;
  return w - o.lr * (mi / o.c1) / (sqrtf(si / o.c2) + o.eps);
}

__device__ __forceinline__ void axpy4(double p, Four q, double (&acc)[4]) {
  acc[0] = fma(p, (double)q.x, acc[0]);
  acc[1] = fma(p, (double)q.y, acc[1]);
  acc[2] = fma(p, (double)q.z, acc[2]);
  acc[3] = fma(p, (double)q.w, acc[3]);
}

// Sums of four values over PARTS neighbouring lanes, scattered: lane `part`
// returns value sum_index<PARTS>(part).
template <int PARTS>
__device__ __forceinline__ double sum4(const double (&v)[4], int part) {
  const bool h = part & (PARTS / 2), l = part & (PARTS / 4);
  const double a = __shfl_xor(h ? v[0] : v[2], PARTS / 2, 64) + (h ? v[2] : v[0]);
  const double b = __shfl_xor(h ? v[1] : v[3], PARTS / 2, 64) + (h ? v[3] : v[1]);
  double s = __shfl_xor(l ? a : b, PARTS / 4, 64) + (l ? b : a);
#pragma unroll
  for (int off = PARTS / 8; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  return s;
}
template <int PARTS>
__device__ __forceinline__ int sum_index(int part) {
  return part / (PARTS / 4);
}

// out[k][a][c] = sum_{i + j = k} sum_b P[i][a][b] Q[j][b][c]   (full
// convolution, Q 5 x 5).  NB / BL lanes, BL values b each, share the sums of
// four consecutive c.
template <int SP, int NA, int NB, int NC, int BL>
__global__ void __launch_bounds__(kStackThreads)
    stack_convolve_kernel(const float* __restrict__ P, const float* __restrict__ Q, float* __restrict__ out) {
  constexpr int SQ = 5, SO = SP + SQ - 1, PARTS = NB / BL;
  const int t = blockIdx.x * kStackThreads + threadIdx.x;
  const int part = t % PARTS, e = t / PARTS;
  if (e >= SO * SO * NA * (NC / 4)) return;
  const int c4 = e % (NC / 4), a = (e / (NC / 4)) % NA, k = e / (NC / 4 * NA);
  const int kq = k / SO, kp = k % SO;
  double acc[4] = {};
  for (int jq = max(0, kq - SP + 1); jq <= min(SQ - 1, kq); ++jq) {
    float p[SQ][BL];
    Four q[SQ][BL];
#pragma unroll
    for (int jp = 0; jp < SQ; ++jp) {
      const int ip = kp - jp;
      const bool in = ip >= 0 && ip < SP;
      const float* pr = P + (((kq - jq) * SP + (in ? ip : 0)) * NA + a) * NB + BL * part;
#pragma unroll
      for (int b = 0; b < BL; ++b) {
        p[jp][b] = in ? pr[b] : 0.f;
        q[jp][b] = *reinterpret_cast<const Four*>(Q + ((jq * SQ + jp) * NB + BL * part + b) * NC + 4 * c4);
      }
    }
#pragma unroll
    for (int jp = 0; jp < SQ; ++jp)
#pragma unroll
      for (int b = 0; b < BL; ++b) axpy4((double)p[jp][b], q[jp][b], acc);
  }
  const double s = sum4<PARTS>(acc, part);
  if (part % (PARTS / 4) == 0) out[4 * e + sum_index<PARTS>(part)] = (float)s;
}

// G12 = out[i][a][b] = sum_j sum_c G[i + j][a][c] Q[j][b][c], Q 5 x 5 with 4
// outputs: one thread per entry, every tap one load of each stack.
__device__ __forceinline__ void correlate_g12(const float* __restrict__ G, const float* __restrict__ Q, int e,
                                              float* __restrict__ out) {
  constexpr int NA = kClosureIn, NB = kClosureHidden, NC = kClosureOut, SG = 13, SQ = 5, SO = SG - SQ + 1;
  static_assert(NC == 4, "one load per tap");
  if (e >= SO * SO * NA * NB) return;
  const int b = e % NB, a = (e / NB) % NA, i = e / (NB * NA);
  const int iq = i / SO, ip = i % SO;
  double acc = 0.0;
#pragma unroll
  for (int jq = 0; jq < SQ; ++jq)
#pragma unroll
    for (int jp = 0; jp < SQ; ++jp)
      acc = dot4(*reinterpret_cast<const Four*>(G + (((iq + jq) * SG + (ip + jp)) * NA + a) * NC),
                 *reinterpret_cast<const Four*>(Q + ((jq * SQ + jp) * NB + b) * NC), acc);
  out[e] = (float)acc;
}

// The third layer's gradient G3[j][b][c] = sum_i sum_a W12[i][a][b] GK[i + j][a][c]
// and its update (blocks 0..24, one tap j each: 32 lanes over b, the taps i over
// 32 slices that meet in LDS), and G12 (the other blocks).
constexpr int kLayer3Threads = 1024;
constexpr int kLayer3Slices = kLayer3Threads / kClosureHidden;
constexpr int kLayer3Blocks12 = (81 * kClosureIn * kClosureHidden + kLayer3Threads - 1) / kLayer3Threads;
__global__ void __launch_bounds__(kLayer3Threads)
    closure_layer3_kernel(const float* __restrict__ W12, const float* __restrict__ GK, const float* __restrict__ W3,
                          float* __restrict__ new3, int off3, Adam opt, float* __restrict__ G12) {
  constexpr int NA = kClosureIn, NB = kClosureHidden, NC = kClosureOut, SP = 9, SG = 13;
  __shared__ double sh[kLayer3Slices][NC][NB];
  if (blockIdx.x >= 25) {
    correlate_g12(GK, W3, (blockIdx.x - 25) * kLayer3Threads + threadIdx.x, G12);
    return;
  }
  const int j = blockIdx.x, jq = j / 5, jp = j % 5;
  const int b = threadIdx.x % NB, slice = threadIdx.x / NB;
  double acc[NC] = {};
  for (int i = slice; i < SP * SP; i += kLayer3Slices) {
    const float* pr = W12 + i * NA * NB + b;
    const float* gr = GK + ((i / SP + jq) * SG + (i % SP + jp)) * NA * NC;
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      axpy4((double)pr[a * NB], reinterpret_cast<const Four*>(gr)[a], acc);
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) sh[slice][c][b] = acc[c];
  __syncthreads();
  if (threadIdx.x >= NB * NC) return;
  const int bo = threadIdx.x / NC, co = threadIdx.x % NC;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < kLayer3Slices; ++k) s += sh[k][co][bo];
  const int e = (j * NB + bo) * NC + co;
  new3[e] = adam_step(opt, off3 + e, W3[e], (float)s);
}

// The first two layers' gradients and updates.  Blocks below kLayer1Blocks:
// G1[i][a][b] = sum_j sum_c G12[i + j][a][c] W2[j][b][c], eight lanes per entry
// with four c each.  The others: G2[j][b][c] = sum_i sum_a W1[i][a][b]
// G12[i + j][a][c], a lane per (four b, c) and tap row iq, the five rows of
// taps meeting in LDS.  The updated layers go to another buffer (new1, new2):
// both gradients read both layers.
constexpr int kLayer1Parts = kClosureHidden / 4;
constexpr int kLayer12Threads = 640;
constexpr int kLayer1Blocks = (25 * kClosureIn * kClosureHidden * kLayer1Parts + kLayer12Threads - 1) / kLayer12Threads;
constexpr int kLayer2Blocks = 50;  // tap j, half of the b groups
__global__ void __launch_bounds__(kLayer12Threads)
    closure_layer12_kernel(const float* __restrict__ W1, const float* __restrict__ W2, const float* __restrict__ G12,
                           float* __restrict__ new1, float* __restrict__ new2, int off1, int off2, Adam opt) {
  constexpr int NA = kClosureIn, NB = kClosureHidden, NC = kClosureHidden, SG = 9;
  __shared__ double sh[5][4][4][NC];
  if (blockIdx.x < kLayer1Blocks) {
    const int t = blockIdx.x * kLayer12Threads + threadIdx.x;
    const int part = t % kLayer1Parts, e = t / kLayer1Parts;
    if (e >= 25 * NA * NB) return;
    const int b = e % NB, a = (e / NB) % NA, i = e / (NB * NA);
    const int iq = i / 5, ip = i % 5;
    double acc = 0.0;
#pragma unroll
    for (int jq = 0; jq < 5; ++jq)
#pragma unroll
      for (int jp = 0; jp < 5; ++jp)
        acc = dot4(reinterpret_cast<const Four*>(G12 + (((iq + jq) * SG + (ip + jp)) * NA + a) * NC)[part],
                   reinterpret_cast<const Four*>(W2 + ((jq * 5 + jp) * NB + b) * NC)[part], acc);
#pragma unroll
    for (int off = kLayer1Parts / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (part == 0) new1[e] = adam_step(opt, off1 + e, W1[e], (float)acc);
    return;
  }
  const int j = (blockIdx.x - kLayer1Blocks) / 2, half = (blockIdx.x - kLayer1Blocks) % 2;
  const int jq = j / 5, jp = j % 5;
  const int c = threadIdx.x % NC, bg = (threadIdx.x / NC) % 4, iq = threadIdx.x / (4 * NC);
  const int b0 = 16 * half + 4 * bg;
  double acc[4] = {};
#pragma unroll
  for (int ip = 0; ip < 5; ++ip)
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const Four p = *reinterpret_cast<const Four*>(W1 + ((iq * 5 + ip) * NA + a) * NB + b0);
      axpy4((double)G12[(((iq + jq) * SG + (ip + jp)) * NA + a) * NC + c], p, acc);
    }
#pragma unroll
  for (int u = 0; u < 4; ++u) sh[iq][bg][u][c] = acc[u];
  __syncthreads();
  if (iq != 0) return;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 5; ++k) s += sh[k][bg][u][c];
    const int e = (j * NB + b0 + u) * NC + c;
    new2[e] = adam_step(opt, off2 + e, W2[e], (float)s);
  }
}

// Gradient of the normalised loss L / yy with respect to the composite
// kernel K (13 x 13 taps):  g[k][ci][co] = 2 (sum_{k', cj} A[k' - k][ci][cj]
// K[k'][cj][co] - C[k][ci][co]) / yy, plus the ridge term 2 rho (K - K0)
// with rho = ridge * (mean zero-offset channel energy) / yy, and per-entry
// terms of the data loss K (R K - 2 C) / yy (summed by closure_loss_kernel).
// One workgroup per tap k, the composite kernel in LDS; sixteen lanes
// (thirteen with work, one k'p each) per ci, the rows k'q over kGradSlices
// groups of lanes that meet in LDS.
constexpr int kGradLanes = 16;
constexpr int kGradSlices = 4;
constexpr int kGradThreads = kClosureIn * kGradLanes * kGradSlices;
__global__ void __launch_bounds__(kGradThreads)
    closure_grad_kernel(const double* __restrict__ stats, const float* __restrict__ K,
                        const float* __restrict__ K0, double ridge, float* __restrict__ g,
                        double* __restrict__ terms) {
  constexpr int NCK = 2 * kClosureHalf + 1, H2 = 2 * kClosureHalf, NA = 2 * H2 + 1;
  constexpr int kRows = (NCK + kGradSlices - 1) / kGradSlices;
  __shared__ Four sk[kClosureKernelElems / 4];
  __shared__ double red[kGradSlices][kClosureIn][kClosureOut];
  const int k = blockIdx.x, tid = threadIdx.x;
  const int k2p = tid % kGradLanes, ci = (tid / kGradLanes) % kClosureIn, slice = tid / (kGradLanes * kClosureIn);
  const int kq = k / NCK, kp = k % NCK;
  const double* A = stats;
  const double* C = stats + kClosureStatsA;
  // this lane's statistics, in flight while the kernel goes to LDS; rows past
  // the end and the three idle lanes take zeros
  double x[kRows][kClosureIn];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int k2q = slice + r * kGradSlices;
    const bool in = k2q < NCK && k2p < NCK;
    const double* ar =
        A + (((in ? k2q - kq + H2 : 0) * NA + (in ? k2p - kp + H2 : 0)) * kClosureIn + ci) * kClosureIn;
#pragma unroll
    for (int cj = 0; cj < kClosureIn; ++cj) x[r][cj] = in ? ar[cj] : 0.0;
  }
  for (int e = tid; e < kClosureKernelElems / 4; e += kGradThreads) sk[e] = reinterpret_cast<const Four*>(K)[e];
  // the values of the last lines, loaded along with the rest
  const int e = k * kClosureIn * kClosureOut + tid % (kClosureIn * kClosureOut);
  const double yy = stats[kClosureStatsA + kClosureStatsC];
  const double c = C[e], ke = (double)K[e], k0 = K0 ? (double)K0[e] : 0.0;
  double mean_diag = 0.0;
#pragma unroll
  for (int cc = 0; cc < kClosureIn; ++cc) mean_diag += A[((H2 * NA + H2) * kClosureIn + cc) * kClosureIn + cc];
  mean_diag /= kClosureIn;
  const double inv = yy > 0.0 ? 1.0 / yy : 0.0;
  __syncthreads();
  double rk[kClosureOut] = {};
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int row = min(slice + r * kGradSlices, NCK - 1) * NCK + min(k2p, NCK - 1);
#pragma unroll
    for (int cj = 0; cj < kClosureIn; ++cj) axpy4(x[r][cj], sk[row * kClosureIn + cj], rk);
  }
  const double part = sum4<kGradLanes>(rk, k2p);
  if (k2p % (kGradLanes / 4) == 0) red[slice][ci][sum_index<kGradLanes>(k2p)] = part;
  __syncthreads();
  if (tid >= kClosureIn * kClosureOut) return;
  double r = 0.0;
#pragma unroll
  for (int w = 0; w < kGradSlices; ++w) r += red[w][tid / kClosureOut][tid % kClosureOut];
  g[e] = (float)(2.0 * (r - c) * inv + 2.0 * ridge * mean_diag * inv * (ke - k0));
  terms[e] = ke * (r - 2.0 * c) * inv;
}

// loss = 1 + sum(terms) (one block, fixed order)
__global__ void closure_loss_kernel(const double* __restrict__ terms, double* __restrict__ loss) {
  __shared__ double red[4];
  double s = 0.0;
  for (int e = threadIdx.x; e < kClosureKernelElems; e += 256) s += terms[e];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *loss = 1.0 + red[0] + red[1] + red[2] + red[3];
}

inline unsigned blocks_for(long long n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

hipError_t launch_closure_weights(const float* K, unsigned short* wb, hipStream_t s) {
  hipLaunchKernelGGL(closure_weights_kernel, dim3(blocks_for(kClosureWeightElems, 256)), dim3(256), 0, s, K, wb);
  return hipGetLastError();
}

template <typename T>
static hipError_t apply_np(int np, const T* v, int level, long long ms, long long ls, long long cs, int nq, int batch,
                           double p0, double dp, const unsigned short* wb, T* out, long long os, hipStream_t s) {
  // one workgroup per CU (its LDS holds the weights and the row ring); each
  // walks about the same number of (member, q group) tasks
  const int tasks = batch * ((nq + kRowsOut - 1) / kRowsOut);
  const unsigned grid = (unsigned)(tasks < 256 ? tasks : 256);
  if (np == 128)
    hipLaunchKernelGGL((closure_apply_kernel<T, 128>), dim3(grid), dim3(kApplyThreads), 0, s, v, level, ms, ls, cs,
                       nq, batch, p0, dp, wb, out, os);
  else if (np == 256)
    hipLaunchKernelGGL((closure_apply_kernel<T, 256>), dim3(grid), dim3(kApplyThreads), 0, s, v, level, ms, ls, cs,
                       nq, batch, p0, dp, wb, out, os);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_closure_apply(int precision, int np, const void* v, int level, long long member_stride,
                                long long level_stride, long long comp_stride, int nq, int batch, double p0,
                                double dp, const unsigned short* wb, void* out, long long out_stride, hipStream_t s) {
  if (precision == QHFPE_FP64)
    return apply_np<double>(np, static_cast<const double*>(v), level, member_stride, level_stride, comp_stride, nq,
                            batch, p0, dp, wb, static_cast<double*>(out), out_stride, s);
  return apply_np<float>(np, static_cast<const float*>(v), level, member_stride, level_stride, comp_stride, nq,
                         batch, p0, dp, wb, static_cast<float*>(out), out_stride, s);
}

// Chunks of rows for a statistics launch: at least kStatWaves rows each, as
// many as the scratch holds, and at most 128 (1536 workgroups, three rounds of
// the GPU, so that the uneven parts even out).
static int stats_chunks(int rows, size_t scratch_bytes) {
  const size_t fit = scratch_bytes / (kStatPartial * sizeof(double));
  long long c = (rows + kStatWaves - 1) / kStatWaves;
  if (c > 128) c = 128;
  if ((size_t)c > fit) c = (long long)fit;
  return (int)c;
}

template <typename T>
static hipError_t stats_np(int np, const T* v, int level, long long ms, long long ls, long long cs, int nq,
                           int batch, double p0, double dp, double* scratch, size_t scratch_bytes, double* stats,
                           hipStream_t s) {
  const int rows = nq * batch;
  int chunks = stats_chunks(rows, scratch_bytes);
  if (chunks < 1) return hipErrorInvalidValue;
  const int per = (rows + chunks - 1) / chunks;
  chunks = (rows + per - 1) / per;
  const dim3 grid(kStatParts, chunks);
  if (np == 128)
    hipLaunchKernelGGL((closure_stats_kernel<T, 128>), grid, dim3(kStatThreads), 0, s, v, level, ms, ls, cs, nq,
                       batch, p0, dp, per, scratch);
  else if (np == 256)
    hipLaunchKernelGGL((closure_stats_kernel<T, 256>), grid, dim3(kStatThreads), 0, s, v, level, ms, ls, cs, nq,
                       batch, p0, dp, per, scratch);
  else
    return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(closure_stats_sum_kernel, dim3(blocks_for(kClosureStatsSize, kSumOutputs)), dim3(4 * kSumOutputs),
                     0, s, scratch, chunks, stats);
  return hipGetLastError();
}

size_t closure_stats_scratch_bytes() { return kStatPartial * sizeof(double); }

hipError_t launch_closure_stats(int precision, int np, const void* v, int level, long long member_stride,
                                long long level_stride, long long comp_stride, int nq, int batch, double p0,
                                double dp, double* scratch, size_t scratch_bytes, double* stats, hipStream_t s) {
  if (precision == QHFPE_FP64)
    return stats_np<double>(np, static_cast<const double*>(v), level, member_stride, level_stride, comp_stride, nq,
                            batch, p0, dp, scratch, scratch_bytes, stats, s);
  return stats_np<float>(np, static_cast<const float*>(v), level, member_stride, level_stride, comp_stride, nq, batch,
                         p0, dp, scratch, scratch_bytes, stats, s);
}

namespace {
using TL = ClosureTrainLayout;

// W12 = W1 * W2 (9 x 9, CI -> M);  K = W12 * W3 (13 x 13, CI -> CO)
hipError_t launch_compose(const float* w, float* st, hipStream_t s) {
  constexpr int CI = kClosureIn, M = kClosureHidden, CO = kClosureOut;
  constexpr int n12 = 81 * CI * (M / 4) * M, nk = 169 * CI * (CO / 4) * M;  // threads
  hipLaunchKernelGGL((stack_convolve_kernel<5, CI, M, M, 1>), dim3(blocks_for(n12, kStackThreads)), dim3(kStackThreads),
                     0, s, w + TL::w1, w + TL::w2, st + TL::w12);
  hipLaunchKernelGGL((stack_convolve_kernel<9, CI, M, CO, 1>), dim3(blocks_for(nk, kStackThreads)), dim3(kStackThreads),
                     0, s, st + TL::w12, w + TL::w3, st + TL::k);
  return hipGetLastError();
}

hipError_t launch_grad(const double* stats, const float* K, const float* prior, double ridge, float* g,
                       double* terms, hipStream_t s) {
  hipLaunchKernelGGL(closure_grad_kernel, dim3(169), dim3(kGradThreads), 0, s, stats, K, prior, ridge, g, terms);
  return hipGetLastError();
}
}  // namespace

// One gradient-descent (Adam) iteration on the three layers; see the layout
// of the training state in qhfpe_internal.hpp.  The layers are read from `from`
// and the updated ones written to `to` (ClosureTrainLayout::w1 or ::g1).
hipError_t launch_closure_train_step(const double* stats, const float* prior, double ridge, float* st, int from,
                                     int to, int t, float lr, hipStream_t s) {
  const float* w = st + from;
  float* wn = st + to;
  hipError_t e = launch_compose(w, st, s);
  if (e != hipSuccess) return e;
  e = launch_grad(stats, st + TL::k, prior, ridge, st + TL::gk, reinterpret_cast<double*>(st + TL::terms), s);
  if (e != hipSuccess) return e;
  Adam opt;
  opt.lr = lr;
  opt.b1 = 0.9f;
  opt.b2 = 0.999f;
  opt.c1 = 1.f - powf(opt.b1, (float)t);
  opt.c2 = 1.f - powf(opt.b2, (float)t);
  opt.eps = 1e-12f;
  opt.m = st + TL::m;
  opt.v = st + TL::v;
  hipLaunchKernelGGL(closure_layer3_kernel, dim3(25 + kLayer3Blocks12), dim3(kLayer3Threads), 0, s, st + TL::w12,
                     st + TL::gk, w + TL::w3, wn + TL::w3, TL::w3, opt, st + TL::g12);
  hipLaunchKernelGGL(closure_layer12_kernel, dim3(kLayer1Blocks + kLayer2Blocks), dim3(kLayer12Threads), 0, s,
                     w + TL::w1, w + TL::w2, st + TL::g12, wn + TL::w1, wn + TL::w2, TL::w1, TL::w2, opt);
  return hipGetLastError();
}

// The normalised data loss of a given composite kernel; terms: scratch of
// kClosureKernelElems doubles, g: scratch of kClosureKernelElems floats.
hipError_t launch_closure_loss(const double* stats, const float* K, float* g, double* terms, double* loss,
                               hipStream_t s) {
  hipError_t e = launch_grad(stats, K, nullptr, 0.0, g, terms, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(closure_loss_kernel, dim3(1), dim3(256), 0, s, terms, loss);
  return hipGetLastError();
}

// The composite kernel of the layers at w1 and its normalised data loss.
hipError_t launch_closure_compose(const double* stats, float* st, double* loss, hipStream_t s) {
  hipError_t e = launch_compose(st, st, s);
  if (e != hipSuccess) return e;
  return launch_closure_loss(stats, st + TL::k, st + TL::gk, reinterpret_cast<double*>(st + TL::terms), loss, s);
}

}  // namespace qhfpe
