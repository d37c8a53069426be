// Pointwise and reduction kernels of the MS-QHFPE library: canonical <->
// packed conversion, dipole commutator, thermal initial state, level-0
// traces, norms and the spectral transforms of Sec. III.
#include <cmath>
#include <mutex>

#include "device_common.hpp"
#include "qhfpe_internal.hpp"

namespace qhfpe {

// Fixed device scratch of the allocation-free entry point (the t3 partial
// sums of the correlation spectrum): every GPU the library runs on holds its
// own copy until the process ends.  Host code never uses this name as an
// address: scratch_pointer() looks the device address up once per device.
static __device__ __align__(256) double scratch[kScratchDoubles];

hipError_t scratch_pointer(double** out) {
  static std::mutex mu;
  static double* ptr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    ptr[dev] = static_cast<double*>(p);
  }
  *out = ptr[dev];
  return hipSuccess;
}

namespace {

// Deterministic block sum / max of one double per thread (kBlock threads).
__device__ double block_sum(double x, double* sh) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  const int tid = threadIdx.x;
  if ((tid & 63) == 0) sh[tid >> 6] = x;
  __syncthreads();
  double s = 0.0;
  if (tid == 0)
    for (int w = 0; w < kBlock / 64; ++w) s += sh[w];
  __syncthreads();
  return s;
}
__device__ double block_max(double x, double* sh) {
  for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off, 64));
  const int tid = threadIdx.x;
  if ((tid & 63) == 0) sh[tid >> 6] = x;
  __syncthreads();
  double s = 0.0;
  if (tid == 0)
    for (int w = 0; w < kBlock / 64; ++w) s = fmax(s, sh[w]);
  __syncthreads();
  return s;
}

// i^(-phase) * (re, im)
__device__ __forceinline__ cx<double> unphase(double re, double im, int phase) {
  switch (phase & 3) {
    case 0: return {re, im};
    case 1: return {im, -re};   // * (-i)
    case 2: return {-re, -im};
    default: return {-im, re};  // * i
  }
}
__device__ __forceinline__ cx<double> dophase(double re, double im, int phase) {
  return unphase(re, im, (4 - (phase & 3)) & 3);
}

// cells of one member: levels * nq * np
template <typename T, int NS>
__global__ void __launch_bounds__(kBlock)
    pack_kernel(GridDesc g, const double* __restrict__ canon, int phase, T* __restrict__ packed,
                int member_offset, double* red) {
  __shared__ double sh[kBlock / 64];
  constexpr int NC = NS * NS;
  const long long cells = (long long)g.levels * g.nq * g.np;
  const int b = blockIdx.y;
  const long long cell = (long long)blockIdx.x * kBlock + threadIdx.x;
  double dev = 0.0, mag = 0.0;
  if (cell < cells) {
    const long long gridn = (long long)g.nq * g.np;
    const int n = (int)(cell / gridn);
    const long long ia = cell % gridn;
    const double* src = canon + (long long)b * g.levels * NC * gridn * 2;
    cx<double> H[NS][NS];
#pragma unroll
    for (int j = 0; j < NS; ++j)
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const long long off = (((long long)(n * NS + j) * NS + k) * gridn + ia) * 2;
        H[j][k] = unphase(src[off], src[off + 1], phase);
        mag = fmax(mag, fabs(H[j][k].re) + fabs(H[j][k].im));
      }
    T* dst = packed + (long long)(member_offset + b) * g.member_stride + (long long)n * g.level_stride + ia;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      dev = fmax(dev, fabs(H[j][j].im));
      dst[j * g.comp_stride] = T(H[j][j].re);
#pragma unroll
      for (int k = j + 1; k < NS; ++k) {
        dev = fmax(dev, fabs(H[j][k].re - H[k][j].re) + fabs(H[j][k].im + H[k][j].im));
        const int c = Packing<NS>::re(j, k);
        dst[c * g.comp_stride] = T(0.5 * (H[j][k].re + H[k][j].re));
        dst[(c + 1) * g.comp_stride] = T(0.5 * (H[j][k].im - H[k][j].im));
      }
    }
  }
  const double d = block_max(dev, sh);
  const double m = block_max(mag, sh);
  if (threadIdx.x == 0) {
    const long long r = ((long long)b * gridDim.x + blockIdx.x) * 2;
    red[r] = d;
    red[r + 1] = m;
  }
}

template <typename T, int NS>
__global__ void __launch_bounds__(kBlock)
    unpack_kernel(GridDesc g, const T* __restrict__ packed, int phase, double* __restrict__ canon,
                  int member_offset) {
  constexpr int NC = NS * NS;
  const long long cells = (long long)g.levels * g.nq * g.np;
  const int b = blockIdx.y;
  const long long cell = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (cell >= cells) return;
  const long long gridn = (long long)g.nq * g.np;
  const int n = (int)(cell / gridn);
  const long long ia = cell % gridn;
  const T* src = packed + (long long)(member_offset + b) * g.member_stride + (long long)n * g.level_stride + ia;
  T h[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) h[c] = src[c * g.comp_stride];
  double* dst = canon + (long long)b * g.levels * NC * gridn * 2;
#pragma unroll
  for (int j = 0; j < NS; ++j)
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const cx<T> e = herm_get<NS>(h, j, k);
      const cx<double> w = dophase((double)e.re, (double)e.im, phase);
      const long long off = (((long long)(n * NS + j) * NS + k) * gridn + ia) * 2;
      dst[off] = w.re;
      dst[off + 1] = w.im;
    }
}

// mu^x on packed H:  W = i^k H -> i^(k+1) H', H' = -i [mu, H]
template <typename T, int NS>
__global__ void __launch_bounds__(kBlock) dipole_kernel(GridDesc g, T* __restrict__ packed, DipoleMu mu) {
  constexpr int NC = NS * NS;
  const long long cells = (long long)g.levels * g.nq * g.np;
  const int b = blockIdx.y;
  const long long cell = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (cell >= cells) return;
  const long long gridn = (long long)g.nq * g.np;
  const int n = (int)(cell / gridn);
  const long long ia = cell % gridn;
  T* p = packed + (long long)b * g.member_stride + (long long)n * g.level_stride + ia;
  T h[NC], o[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) h[c] = p[c * g.comp_stride];
  T A[NS][NS];
#pragma unroll
  for (int j = 0; j < NS; ++j)
#pragma unroll
    for (int k = 0; k < NS; ++k) A[j][k] = T(mu.m[j][k]);
  commutator_mi<NS, T>(A, h, o);
#pragma unroll
  for (int c = 0; c < NC; ++c) p[c * g.comp_stride] = o[c];
}

template <typename T, int NS>
__global__ void __launch_bounds__(kBlock)
    thermal_kernel(GridDesc g, T* __restrict__ packed, double q0, double dq, double p0, double dp,
                   const double* __restrict__ bath, double omega, double mass, double hbar,
                   const double* __restrict__ noise) {
  constexpr int NC = NS * NS;
  const long long gridn = (long long)g.nq * g.np;
  const long long cells = (long long)g.levels * gridn;
  const int b = blockIdx.y;
  const long long cell = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (cell >= cells) return;
  const int n = (int)(cell / gridn);
  const long long ia = cell % gridn;
  T* p = packed + (long long)b * g.member_stride + (long long)n * g.level_stride + ia;
  double w = 0.0;
  if (n == 0) {
    // b = beta hbar omega / 2 with this member's beta
    const double tanh_b = tanh(0.5 * bath[kBathStride * b + 4] * hbar * omega);
    const int i = (int)(ia / g.np), a = (int)(ia % g.np);
    const double q = q0 + i * dq, pp = p0 + a * dp;
    w = (tanh_b / (M_PI * hbar)) *
        exp(-tanh_b * (pp * pp / (mass * hbar * omega) + mass * omega * q * q / hbar));
    if (noise) w += noise[ia];
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) p[c * g.comp_stride] = T(c == 0 ? w : 0.0);
}

// Level-0 trace partials with the same tiling as the stage kernel: one wave
// per tile.
template <typename T, int NS>
__global__ void __launch_bounds__(kBlock)
    trace_kernel(GridDesc g, const T* __restrict__ packed, DipoleMu mu, int tq, int ntiles,
                 double* __restrict__ partials) {
  const int lane = threadIdx.x & 63;
  const int tile = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6), b = blockIdx.y;
  if (tile >= ntiles) return;
  const T* p = packed + (long long)b * g.member_stride;
  const int cells = min(tq, g.nq - tile * tq) * g.np;
  double tr = 0.0;
  for (int e = lane; e < cells; e += 64) {
    const long long ia = (long long)tile * tq * g.np + e;
#pragma unroll
    for (int j = 0; j < NS; ++j) tr += mu.m[j][j] * (double)p[j * g.comp_stride + ia];
#pragma unroll
    for (int j = 0; j < NS; ++j)
#pragma unroll
      for (int k = j + 1; k < NS; ++k)
        tr += 2.0 * mu.m[j][k] * (double)p[Packing<NS>::re(j, k) * g.comp_stride + ia];
  }
  for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off, 64);
  if (lane == 0) partials[(long long)b * ntiles + tile] = tr;
}

// One wave per response sample: its lanes sum the partials (lane by lane in
// order, then a butterfly).
__global__ void __launch_bounds__(kBlock)
    finalize_kernel(int ntiles, int nslots, const double* __restrict__ partials, long long slot_stride, double scale,
                    int phase, double* __restrict__ resp, long long resp_stride, long long resp_offset, int* flag) {
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const int b = blockIdx.y;
  if (j >= nslots) return;
  const double* p = partials + j * slot_stride + (long long)b * ntiles;
  double s = 0.0;
  for (int t = lane; t < ntiles; t += 64) s += p[t];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane != 0) return;
  s *= scale;
  const cx<double> w = dophase(s, 0.0, phase);
  if (resp) {
    double* r = resp + (long long)b * resp_stride + (resp_offset + j) * 2;
    r[0] = w.re;
    r[1] = w.im;
  }
  if (!isfinite(s)) *flag = 1;
}

template <typename T, int NC>
__global__ void __launch_bounds__(kBlock)
    norm_kernel(GridDesc g, const T* __restrict__ packed, int ns, double* __restrict__ red) {
  __shared__ double sh[kBlock / 64];
  const long long gridn = (long long)g.nq * g.np;
  const long long cells = (long long)g.levels * gridn;
  const int b = blockIdx.y;
  double s = 0.0;
  for (long long cell = (long long)blockIdx.x * kBlock + threadIdx.x; cell < cells;
       cell += (long long)gridDim.x * kBlock) {
    const int n = (int)(cell / gridn);
    const long long ia = cell % gridn;
    const T* p = packed + (long long)b * g.member_stride + (long long)n * g.level_stride + ia;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double x = (double)p[c * g.comp_stride];
      // off-diagonal packed entries stand for two canonical entries
      s += (c < ns ? 1.0 : 2.0) * x * x;
    }
  }
  const double t = block_sum(s, sh);
  if (threadIdx.x == 0) red[(long long)b * gridDim.x + blockIdx.x] = t;
}

// ---------------------------------------------------------------------------
// Spectral sums of Sec. III.  The phase factors exp(i omega s dt) of
// consecutive samples differ by one rotation, so a thread evaluates sincos
// once per kPhaseChunk * kPhaseRestart samples of its omega and rotates in
// between (four operations a sample; one sincos takes about a hundred).  Two
// levels keep the rotations' rounding small: a chunk's samples are rotated
// from the chunk's first factor, the chunks' first factors from the last
// sincos, so no factor is more than kPhaseChunk + kPhaseRestart rotations away
// from a sincos (2e-15; the product omega * s * dt itself rounds at 1e-16 of
// a phase that reaches several hundred).
// ---------------------------------------------------------------------------
constexpr int kPhaseChunk = 16;
constexpr int kPhaseRestart = 8;
constexpr int kSpectrumThreads = 1024;

struct Phase {
  double re, im;
};
__device__ __forceinline__ Phase phase_of(double x) {
  Phase p;
  sincos(x, &p.im, &p.re);
  return p;
}
__device__ __forceinline__ Phase rotate(Phase a, Phase b) {
  return {fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re)};
}

// one complex sample (aligned as a double: callers' series need not be
// aligned to 16 bytes)
struct Sample {
  double re, im;
};

// sum_{s = s0}^{s1 - 1} c_s Im(e^{i om s dt} x[s]) of a series of n samples, c_s
// the trapezoid weights
__device__ __forceinline__ double phase_sum(const Sample* __restrict__ x, long long n, long long s0, long long s1,
                                            double om, double dt) {
  const Phase e1 = phase_of(om * dt), ec = phase_of(om * (double)kPhaseChunk * dt);
  Phase base = {1.0, 0.0};
  double acc = 0.0;
  int k = 0;
  for (long long c = s0; c < s1; c += kPhaseChunk, ++k) {
    base = (k % kPhaseRestart == 0) ? phase_of(om * (double)c * dt) : rotate(base, ec);
    Phase e = base;
    if (c > 0 && c + kPhaseChunk <= s1 && c + kPhaseChunk < n) {
#pragma unroll
      for (int j = 0; j < kPhaseChunk; ++j) {
        const Sample v = x[c + j];
        acc = fma(e.im, v.re, fma(e.re, v.im, acc));
        if (j + 1 < kPhaseChunk) e = rotate(e, e1);
      }
    } else {
      // a chunk with an end of the series, or a partial one
      for (long long s = c; s < min(s1, c + kPhaseChunk); ++s) {
        const double g = (s == 0 || s == n - 1) ? 0.5 : 1.0;
        const Sample v = x[s];
        acc = fma(g * e.im, v.re, fma(g * e.re, v.im, acc));
        e = rotate(e, e1);
      }
    }
  }
  return acc;
}

// samples per segment when n samples are split into at most `segs` segments
// of whole chunks
__host__ __device__ __forceinline__ long long segment_length(long long n, int segs) {
  const long long l = (n + segs - 1) / segs;
  return (l + kPhaseChunk - 1) / kPhaseChunk * kPhaseChunk;
}

// out[w] = omega_w dt sum_s c_s Im(e^{i omega_w s dt} R[s]).  Bound by FP64
// issue and by how many CUs take part: a workgroup owns `wpb` frequencies and
// splits the samples over blockDim / wpb segments, whose sums meet in LDS
// (no scratch memory, fixed order).  20001 samples at 2001 frequencies take
// 23 us a call; one thread per frequency over all samples with a sincos per
// sample took 4430 us.
__global__ void __launch_bounds__(kSpectrumThreads)
    spectrum_abs_kernel(const Sample* __restrict__ series, long long n, double dt, const double* __restrict__ omega,
                        int n_omega, int wpb, double* __restrict__ out) {
  __shared__ double sh[kSpectrumThreads];
  const int tid = threadIdx.x, segs = blockDim.x / wpb;
  const int seg = tid / wpb, w = blockIdx.x * wpb + tid % wpb;
  const double om = omega[min(w, n_omega - 1)];
  const long long len = segment_length(n, segs);
  const long long s0 = seg * len, s1 = min(n, s0 + len);
  sh[tid] = s0 < s1 ? phase_sum(series, n, s0, s1, om, dt) : 0.0;
  for (int half = segs / 2; half > 0; half /= 2) {
    __syncthreads();
    if (seg < half) sh[tid] += sh[tid + half * wpb];
  }
  if (seg == 0 && w < n_omega) out[w] = om * sh[tid] * dt;
}

// im[t1][w3] = Im sum_t3 c dt3 e^{i w3 t3} R3[t1][t3], the part of the t3 sums
// that the spectrum needs: a contraction over t3, on the FP64 matrix cores
// (v_mfma_f64_16x16x4: rows t1, columns w3, four samples).  A workgroup holds a
// 16 x 16 tile; its sixteen waves take a segment of the samples each and meet in
// LDS, and where the tiles leave CUs idle two workgroups share a tile's samples
// (partial sums im[0], im[1], which the next kernel adds).  Of eight samples a
// step, lane (k, column) rotates the factors of samples 2 k, 2 k + 1, which serve
// sixteen rows; the samples come in blocks of whole 512-byte row pieces and change
// lanes in LDS (loaded by the lanes that multiply them, 64 cache lines a load, the
// kernel takes 27 us).  64 x 4001 samples at 401 frequencies take 20 us
// (7 of them matrix issue); on the vector units with scalar sample loads,
// bound by those loads, they took 38 us, and with one thread per (t1, frequency)
// and a sincos per sample the two passes took 1180 us.
constexpr int kCorrWaves = kSpectrumThreads / 64;
constexpr int kCorrTile = 16;
constexpr int kCorrStep = 8;     // samples per step
constexpr int kCorrSpan = 32;    // samples per block: one load brings two rows of it
constexpr int kCorrRestart = 4;  // blocks between sincos: factors at most 16 rotations from one
constexpr int kCorrRow = kCorrSpan + 1;  // padded LDS row (in samples)
typedef double f64x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(kSpectrumThreads)
    spectrum_corr_t3_kernel(const Sample* __restrict__ r3, int n1, int n3, double dt3,
                            const double* __restrict__ w3, int nw3, int planes, double* __restrict__ im) {
  typedef double pair __attribute__((ext_vector_type(2)));
  __shared__ pair slab[kCorrWaves][kCorrTile * kCorrRow];  // per wave: a block of its rows
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, k = lane >> 4;
  const int row0 = blockIdx.y * kCorrTile, col0 = blockIdx.x * kCorrTile;
  // (rows and columns past the edges repeat the last one and are not stored)
  const double om = w3[min(col0 + li, nw3 - 1)];
  const int segs = kCorrWaves * planes, seg = wid * planes + (int)blockIdx.z;
  const int per = ((n3 + segs - 1) / segs + kCorrStep - 1) / kCorrStep * kCorrStep;
  const long long s0 = (long long)seg * per;
  const int len = (int)max(0ll, min((long long)per, n3 - s0));  // this wave's samples
  constexpr int kLoads = kCorrTile / 2;
  const int half = lane / kCorrSpan, ls = lane % kCorrSpan;  // of a load: this lane's row and sample
  auto load = [&](int at, Sample (&v)[kLoads]) {
    const long long s = min(s0 + at + ls, (long long)n3 - 1);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) v[i] = r3[(long long)min(row0 + 2 * i + half, n1 - 1) * n3 + s];
  };
  Sample next[kLoads];
  if (len > 0) load(0, next);
  const Phase e1 = phase_of(om * dt3), e8 = phase_of(om * (double)kCorrStep * dt3);
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  Phase e = {1.0, 0.0};
  for (int at = 0, blk = 0; at < len; at += kCorrSpan, ++blk) {
    // into LDS with the trapezoid weights of the ends, zero past the segment
    const bool used = at + ls < len;
    const double g = (s0 + at + ls == 0 || s0 + at + ls == n3 - 1) ? 0.5 : 1.0;
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < kLoads; ++i)
      slab[wid][(2 * i + half) * kCorrRow + ls] = pair{used ? g * next[i].re : 0.0, used ? g * next[i].im : 0.0};
    wave_lds_sync();
    load(at + kCorrSpan, next);  // (past the end: the rows' last samples, not used)
    if (blk % kCorrRestart == 0) e = phase_of(om * (double)(s0 + at + 2 * k) * dt3);
#pragma unroll
    for (int t = 0; t < kCorrSpan / kCorrStep; ++t) {
      const pair* const z = slab[wid] + li * kCorrRow + kCorrStep * t + 2 * k;
      const pair u = z[0], v = z[1];
      const Phase f = rotate(e, e1);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(u[0], e.im, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(u[1], e.re, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0], f.im, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1], f.re, acc, 0, 0, 0);
      e = rotate(e, e8);
    }
  }
  // D layout of the FP64 product: row 4 r + lane / 16, column lane % 16
  double* const mine = reinterpret_cast<double*>(slab[wid]);
  wave_lds_sync();
#pragma unroll
  for (int r = 0; r < 4; ++r) mine[(4 * r + k) * kCorrTile + li] = acc[r];
  __syncthreads();
  if (tid < kCorrTile * kCorrTile) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kCorrWaves; ++w) s += reinterpret_cast<const double*>(slab[w])[tid];
    const int r = row0 + tid / kCorrTile, w = col0 + tid % kCorrTile;
    if (r < n1 && w < nw3) im[((long long)blockIdx.z * n1 + r) * nw3 + w] = s * dt3;
  }
}

// out[w3][w1] = sum_t1 c dt1 2 cos(w1 t1) Im A[t1][w3]: a lane holds one w1 and
// kCorrRows frequencies w3, which share the cosine; the waves of a workgroup
// take every kWaves-th chunk of coherence times (whose sums, the same for the
// whole wave, come through scalar loads issued together: as many as the scalar
// registers hold) and meet in LDS.  10 us for 64 coherence times at 401 x 401
// frequencies in two planes (13 with sixteen waves); 21 us for one plane as one
// wave per workgroup with loads one by one.
constexpr int kCorrRows = 4;
constexpr int kCorrT1Waves = 8;
template <int PLANES>
__global__ void __launch_bounds__(64 * kCorrT1Waves)
    spectrum_corr_t1_kernel(const double* __restrict__ im, int n1, double dt1, const double* __restrict__ w1,
                            int nw1, int nw3, double* __restrict__ out) {
  constexpr int kWaves = kCorrT1Waves, kChunk = 8 / PLANES;
  __shared__ double sh[kWaves][kCorrRows][64];
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w0 = blockIdx.y * kCorrRows;
  const double om = w1[min((int)blockIdx.x * 64 + lane, nw1 - 1)];
  const Phase e1 = phase_of(om * dt1);
  double acc[kCorrRows] = {};
  for (int c = wid * kChunk; c < n1; c += kWaves * kChunk) {
    double x[kChunk][kCorrRows][PLANES];
#pragma unroll
    for (int j = 0; j < kChunk; ++j)
#pragma unroll
      for (int r = 0; r < kCorrRows; ++r)
#pragma unroll
        for (int u = 0; u < PLANES; ++u)
          x[j][r][u] = im[((long long)u * n1 + min(c + j, n1 - 1)) * nw3 + min(w0 + r, nw3 - 1)];
    Phase e = phase_of(om * (double)c * dt1);
#pragma unroll
    for (int j = 0; j < kChunk; ++j) {
      const int s = c + j;
      if (s < n1) {
        const double g = (s == 0 || s == n1 - 1) ? e.re : 2.0 * e.re;
#pragma unroll
        for (int r = 0; r < kCorrRows; ++r)
          acc[r] = fma(g, PLANES == 2 ? x[j][r][0] + x[j][r][PLANES - 1] : x[j][r][0], acc[r]);
      }
      e = rotate(e, e1);
    }
  }
#pragma unroll
  for (int r = 0; r < kCorrRows; ++r) sh[wid][r][lane] = acc[r];
  __syncthreads();
  // wave r sums frequency row r
  const int r = wid, a = blockIdx.x * 64 + lane;
  if (r >= kCorrRows || w0 + r >= nw3 || a >= nw1) return;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) s += sh[k][r][lane];
  out[(long long)(w0 + r) * nw1 + a] = s * dt1;
}

__global__ void clear_flag_kernel(int* flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *flag = 0;
}

// Streaming device copy: every lane moves kCopyUnroll 16-byte vectors, all
// loads issued before the first store, consecutive lanes on consecutive
// vectors (each load and store instruction of a wave covers 1 KiB).
constexpr int kCopyUnroll = 4;
__global__ void __launch_bounds__(kBlock)
    stream_copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, long long n16) {
  const long long base = (long long)blockIdx.x * (kBlock * kCopyUnroll) + threadIdx.x;
  uint4 v[kCopyUnroll];
#pragma unroll
  for (int k = 0; k < kCopyUnroll; ++k) {
    const long long i = base + (long long)k * kBlock;
    if (i < n16) v[k] = src[i];
  }
#pragma unroll
  for (int k = 0; k < kCopyUnroll; ++k) {
    const long long i = base + (long long)k * kBlock;
    if (i < n16) dst[i] = v[k];
  }
}

// the bytes past the last whole 16-byte vector (fewer than 16)
__global__ void copy_tail_kernel(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst, int n) {
  const int i = threadIdx.x;
  if (i < n) dst[i] = src[i];
}

inline dim3 cell_grid(const GridDesc& g, int nmembers) {
  const long long cells = (long long)g.levels * g.nq * g.np;
  return dim3((unsigned)((cells + kBlock - 1) / kBlock), (unsigned)nmembers);
}

}  // namespace

#define QHFPE_DISPATCH(g, F)                                  \
  do {                                                        \
    if ((g).precision == QHFPE_FP64) {                        \
      if ((g).ns == 2) { F(double, 2); } else { F(double, 3); } \
    } else {                                                  \
      if ((g).ns == 2) { F(float, 2); } else { F(float, 3); }   \
    }                                                         \
  } while (0)

hipError_t launch_pack(const GridDesc& g, const double* canon, int phase, void* packed, int member_offset,
                       int nmembers, double* red, int* nred_blocks, hipStream_t s) {
  const dim3 grid = cell_grid(g, nmembers);
  *nred_blocks = (int)grid.x;
#define F(T, NS) hipLaunchKernelGGL((pack_kernel<T, NS>), grid, dim3(kBlock), 0, s, g, canon, phase, \
                                    static_cast<T*>(packed), member_offset, red)
  QHFPE_DISPATCH(g, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_unpack(const GridDesc& g, const void* packed, int phase, double* canon, int member_offset,
                         int nmembers, hipStream_t s) {
  const dim3 grid = cell_grid(g, nmembers);
#define F(T, NS) hipLaunchKernelGGL((unpack_kernel<T, NS>), grid, dim3(kBlock), 0, s, g, \
                                    static_cast<const T*>(packed), phase, canon, member_offset)
  QHFPE_DISPATCH(g, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_dipole(const GridDesc& g, void* packed, const double mu[3][3], hipStream_t s) {
  const dim3 grid = cell_grid(g, g.batch);
  DipoleMu m;
  for (int j = 0; j < 3; ++j)
    for (int k = 0; k < 3; ++k) m.m[j][k] = mu[j][k];
#define F(T, NS) hipLaunchKernelGGL((dipole_kernel<T, NS>), grid, dim3(kBlock), 0, s, g, static_cast<T*>(packed), m)
  QHFPE_DISPATCH(g, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_thermal(const GridDesc& g, void* packed, double q0, double dq, double p0, double dp,
                          const double* bath, double omega, double mass, double hbar, const double* noise,
                          hipStream_t s) {
  const dim3 grid = cell_grid(g, g.batch);
#define F(T, NS) hipLaunchKernelGGL((thermal_kernel<T, NS>), grid, dim3(kBlock), 0, s, g, static_cast<T*>(packed), \
                                    q0, dq, p0, dp, bath, omega, mass, hbar, noise)
  QHFPE_DISPATCH(g, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_trace_partials(const GridDesc& g, const void* packed, const double mu[3][3], int tq,
                                 int ntiles, double* partials, hipStream_t s) {
  DipoleMu m;
  for (int j = 0; j < 3; ++j)
    for (int k = 0; k < 3; ++k) m.m[j][k] = mu[j][k];
  const dim3 grid((ntiles + kBlock / 64 - 1) / (kBlock / 64), g.batch);
#define F(T, NS) hipLaunchKernelGGL((trace_kernel<T, NS>), grid, dim3(kBlock), 0, s, g, \
                                    static_cast<const T*>(packed), m, tq, ntiles, partials)
  QHFPE_DISPATCH(g, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_finalize(int batch, int ntiles, int nslots, const double* partials, long long slot_stride,
                           double scale, int phase, double* resp, long long resp_stride, long long resp_offset, int* flag,
                           hipStream_t s) {
  const dim3 grid((nslots + kBlock / 64 - 1) / (kBlock / 64), batch);
  hipLaunchKernelGGL(finalize_kernel, grid, dim3(kBlock), 0, s, ntiles, nslots, partials, slot_stride, scale,
                     phase, resp, resp_stride, resp_offset, flag);
  return hipGetLastError();
}

hipError_t launch_norm_partials(const GridDesc& g, const void* packed, double* red, int* nblocks_per_member,
                                hipStream_t s) {
  const long long cells = (long long)g.levels * g.nq * g.np;
  int nb = (int)((cells + kBlock - 1) / kBlock);
  if (nb > 1024) nb = 1024;
  *nblocks_per_member = nb;
  const dim3 grid(nb, g.batch);
#define F(T, NS) hipLaunchKernelGGL((norm_kernel<T, NS * NS>), grid, dim3(kBlock), 0, s, g, \
                                    static_cast<const T*>(packed), NS, red)
  QHFPE_DISPATCH(g, F);
#undef F
  return hipGetLastError();
}

hipError_t launch_clear_flag(int* flag, hipStream_t s) {
  hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(64), 0, s, flag);
  return hipGetLastError();
}

hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  if ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) % 16) return hipErrorInvalidValue;
  const long long n16 = (long long)(bytes / 16);
  const int tail = (int)(bytes % 16);
  if (n16 > 0) {
    const long long per_block = (long long)kBlock * kCopyUnroll;
    const long long blocks = (n16 + per_block - 1) / per_block;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(stream_copy_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       static_cast<const uint4*>(src), static_cast<uint4*>(dst), n16);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (tail) {
    hipLaunchKernelGGL(copy_tail_kernel, dim3(1), dim3(64), 0, s, static_cast<const unsigned char*>(src) + 16 * n16,
                       static_cast<unsigned char*>(dst) + 16 * n16, tail);
    return hipGetLastError();
  }
  return hipSuccess;
}

hipError_t launch_spectrum_abs(const double* series, long long n, double dt, const double* omega, int n_omega,
                               double* out, hipStream_t s) {
  // frequencies per workgroup: about one workgroup per CU, 4 to 64 (a
  // frequency's samples then split over up to 256 segments); segments: a
  // power of two, at least two chunks of samples each
  int wpb = 4;
  while (wpb < 64 && n_omega > 256 * wpb) wpb *= 2;
  int segs = 64 / wpb > 1 ? 64 / wpb : 1;
  while (segs * wpb * 2 <= kSpectrumThreads && n >= (long long)segs * 4 * kPhaseChunk) segs *= 2;
  hipLaunchKernelGGL(spectrum_abs_kernel, dim3((n_omega + wpb - 1) / wpb), dim3(wpb * segs), 0, s,
                     reinterpret_cast<const Sample*>(series), n, dt, omega, n_omega, wpb, out);
  return hipGetLastError();
}

hipError_t launch_spectrum_corr(const double* r3, int n1, int n3, double dt1, double dt3, const double* w1,
                                int nw1, const double* w3, int nw3, double* work, double* out, hipStream_t s) {
  // d_work holds two planes; with a workgroup per CU (256 tiles) one is enough
  const dim3 tiles((nw3 + kCorrTile - 1) / kCorrTile, (n1 + kCorrTile - 1) / kCorrTile);
  const int planes = (long long)tiles.x * tiles.y < 256 ? 2 : 1;
  hipLaunchKernelGGL(spectrum_corr_t3_kernel, dim3(tiles.x, tiles.y, planes), dim3(kSpectrumThreads), 0, s,
                     reinterpret_cast<const Sample*>(r3), n1, n3, dt3, w3, nw3, planes, work);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid((nw1 + 63) / 64, (nw3 + kCorrRows - 1) / kCorrRows), block(64 * kCorrT1Waves);
  if (planes == 2)
    hipLaunchKernelGGL(spectrum_corr_t1_kernel<2>, grid, block, 0, s, work, n1, dt1, w1, nw1, nw3, out);
  else
    hipLaunchKernelGGL(spectrum_corr_t1_kernel<1>, grid, block, 0, s, work, n1, dt1, w1, nw1, nw3, out);
  return hipGetLastError();
}

}  // namespace qhfpe
