// Internal declarations shared by the host API and the kernels of the
// MS-QHFPE library.  Not part of the public C-ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "qhfpe.h"

namespace qhfpe {

constexpr int kBlock = 256;        // threads per workgroup of every grid kernel
// Response samples buffered between finalisations: as many as kPartialBytes of
// trace partials hold, but at least kMinRespSlots (a batch of many members then
// holds at most 128 bytes of partials per column and member, 8% of the smallest
// state) and at most kMaxRespSlots.
constexpr int kMaxRespSlots = 256, kMinRespSlots = 16;
constexpr size_t kPartialBytes = size_t(2) << 20;
constexpr int kBathStride = 8;     // doubles per member in the bath table

// Two-pass FFT plan along p (np = n1 * n2, n1 even) for every supported np.
struct Plan {
  int np, n1, n2;
};
constexpr Plan kPlans[] = {
    {8, 4, 2},   {12, 4, 3},  {16, 4, 4},   {24, 6, 4},    {32, 8, 4},    {48, 8, 6},
    {64, 8, 8},  {96, 12, 8}, {128, 16, 8}, {192, 16, 12}, {256, 16, 16},
};
inline const Plan* find_plan(int np) {
  for (const Plan& p : kPlans)
    if (p.np == np) return &p;
  return nullptr;
}
// The wave variant's plan: the same but at np = 96, where its first pass takes 8
// points (a wave's 64 lanes hold whole transforms of the second pass, which
// has np / 8 = 12 of them) and the workgroup variant's 12 (three states with
// q-dependent couplings, 96 x 96 x 5, 16 members: FP32 38.1 us a stage against 41.1
// with 8, FP64 80.7 against 86.4; two states, code 2: 14.0 / 15.5, 21.9 / 23.2).
constexpr int wave_n1(int np) { return np == 96 ? 8 : np <= 24 ? 0 : np <= 64 ? 8 : 16; }

// Stage workgroup shape: G = max(1, 256/np) groups of np threads; each
// thread owns one p node of CPT consecutive q columns; a tile is TQ = G*CPT
// columns (even, so three-state tiles can pair columns).  CPT is a tuning
// variant: 2, 4 or 8 for FP32 two-state; 2 or 4 for FP64 two-state and FP32
// three-state; 2 for FP64 three-state (larger LDS tiles would not fit).
constexpr int plan_groups(int np) { return np >= 256 ? 1 : 256 / np; }
constexpr int kMinCpt = 2;
// The workgroup variant with a q-dependent coupling (the coupling surfaces
// in the r-space multiply) exists for 2 cells per thread only.
constexpr int kQcCpt = 2;
constexpr bool cpt_supported_c(int elem_bytes, int ns, int cpt) {
  return (ns == 2) ? (cpt == 2 || cpt == 4 || (cpt == 8 && elem_bytes == 4))
                   : (elem_bytes == 8 ? cpt == 2 : (cpt == 2 || cpt == 4));
}
inline bool cpt_supported(int elem_bytes, int ns, int cpt) { return cpt_supported_c(elem_bytes, ns, cpt); }
// Three states: 2 cells per thread in both precisions (with 4, the LDS of a
// 256-thread workgroup leaves room for one workgroup per CU at np = 256).
inline int cpt_default(int /*elem_bytes*/, int ns) { return (ns == 3) ? 2 : 4; }

// Tile code of the wave-independent stage variant (stage_wave.hpp) at np = 128
// and 256; at the other np that it covers it computes the default code.
constexpr int kTileWave = 1;
constexpr int kMaxGroups = 4;  // member groups (streams) of qhfpe_step
// Multiplier planes of the wave variant: two states 5, three states 6.
constexpr int kWaveTables = 5;
constexpr int kWaveTables3 = 6;
inline int wave_table_planes(int ns) { return ns == 3 ? kWaveTables3 : kWaveTables; }
// p nodes per lane of the wave variant (a column lies on np / wave_nodes
// lanes: 16, 32 or 64); 0 where it does not exist.  Several nodes a lane make
// wide loads and few lane exchanges; 64 takes one so that a column fills the wave.
constexpr int wave_nodes(int np) {
  return np == 256 ? 4 : (np == 192 || np == 96 || np == 48) ? 3 : (np == 128 || np == 32) ? 2 : np == 64 ? 1 : 0;
}
constexpr bool wave_exists(int np) { return wave_nodes(np) != 0; }
// public tile code 1
inline bool wave_supported(int ns, int np) { return ns == 2 && (np == 128 || np == 256); }
inline bool wave_variant_supported(int /*elem_bytes*/, int /*ns*/, int np) { return np == 128 || np == 256; }
// the workgroup variant with a q-dependent coupling: not where the two-state wave
// variant computes its tile code
constexpr bool workgroup_qc(int ns, int np) { return ns == 3 || !wave_exists(np) || np == 128 || np == 256; }
// Shape of a wave launch: q columns per lane group, components in flight (or
// kStaggered), waves per workgroup.
constexpr int kStaggered = 0;
struct WaveShape {
  int c = 0, pf = 0, wpb = 0;
};
constexpr int wave_groups(int np) { return 64 * wave_nodes(np) / np; }  // lane groups per wave
inline int wave_columns_of(int np, int c) { return wave_groups(np) * c; }

// The shape for a handle whose stages would be `waves` waves with one column
// per lane group; launched in member groups, `spread` is the count of groups
// times the largest one's waves (else `waves`).  Results do not depend on it.  One column per wave keeps a
// wave's chain short (few loads to wait for, one item per FFT round) but loads
// 7 window columns per column and leaves FFT lanes idle: it wins while the
// waves find SIMDs of their own.  More columns per wave save loads and fill
// the FFT rounds, which wins once several waves share a SIMD.  Measured (us
// per stage launch, one column / two / four per lane group):
//   two states: 128 FP64, 896 waves 7.6 / 7.9 / 10.6, 2688 waves 11.2 / 10.6 /
//   -, 7168 waves 21 / 17.5 / 17.4, 28672 waves 97 / 81 / 73; 64 FP32, 1280
//   waves 6.2 / 6.5 / 8.1, 10240 waves 14.3 / 10.9 / 10.2; 256 FP64, 192 waves
//   9.0 / 10.1, 2304 waves 21.2 / 18.2; 96 FP64 (two lane groups), 1344 waves
//   10.3 / 11.4, 5376 waves 23.5 / 19.8 / 32.7.
//   128 FP32, two / four columns: one launch 10000 waves 16.7 / 16.4, 10500 18.1 /
//   16.5; two groups of 8 members each 10000 14.4 / 15.4, 11000 15.8 / 15.6; five
//   members (three and two) 8500 waves 13.1 / 14.6, 9000 15.2 / 14.6.
//   three states: 128 FP32, one launch 7700 waves 32.1 / 32.8, 8400 34.9 / 34.6, 9600
//   39.7 / 35.9; in groups, whose launches overlap, sooner: 16 members 4400 waves
//   17.8 / 18.1, 5000 19.4 / 18.7, 9600 35.2 / 30.4; 128 FP64, one launch 10500 75.6 /
//   77.8, 11500 87.4 / 85.0, in groups five members 3800 24.3 / 24.5, 4400 29.4 / 27.0;
//   64 FP64, 11520 waves 41.8 / 36.6; 256 FP32, 9216 waves 55.6 with one (two would
//   leave LDS for six waves a CU).
// Components in flight: with SIMDs to spare a one-column wave issues two (three
// for nine components; in FP32 all four of two states: 64 x 64 5.2 against
// 5.3 us); otherwise the staggered schedule, except FP32 at 256, whose second
// register slots would cost it the fourth wave per SIMD (14.2 against 15.1 us).
// Workgroups: two waves spread more evenly over the CUs, four share the tables
// (256 FP64 1152 tasks 18.2 against 21.4 us, 9216 tasks 111 against 105 us;
// at 192 four win throughout).
inline WaveShape wave_shape(int elem_bytes, int ns, int np, bool qcoup, long long waves, long long spread, bool grouped,
                            bool stream) {
  const bool f32 = elem_bytes == 4;
  if (ns == 3) {
    const bool pairs = np == 128 || np == 64;  // two columns fit
    const long long two = np == 64 ? 7000 : grouped ? 4700 : f32 ? 8400 : 11000;
    if (pairs && (stream || (np == 64 ? waves : spread) >= two)) return {2, kStaggered, 2};
    if ((f32 || pairs) && !stream && waves <= 2000) return {1, 3, 1};
    return {1, kStaggered, 2};
  }
  if (!stream && waves <= (wave_groups(np) > 1 ? 2800 : 1400)) {
    if (f32 && !qcoup && waves <= 700) return {1, 4, 1};
    return {1, 2, 1};
  }
  if (np == 256) {
    const int pf = f32 && !qcoup ? 1 : kStaggered;
    return {2, pf, stream || waves > 7000 ? 4 : 2};
  }
  if (np == 192) return {2, kStaggered, 4};
  if (np == 128 && (stream || waves >= 13000 || (f32 && !qcoup && spread >= 10300))) return {4, kStaggered, 4};
  if (np == 64 && (stream || waves >= 7000)) return {4, kStaggered, 4};
  return {2, kStaggered, 2};
}

// Exact division of 0 <= t < 2^31 by a fixed d >= 1 with one high product
// (round-up method: 2^(32 + s) / d with s = ceil(log2 d), the 2^32 of the
// multiplier added by hand).
struct FixedDiv {
  unsigned mul = 0;
  int shift = 0;
  static FixedDiv by(unsigned d) {
    FixedDiv f;
    while ((1ull << f.shift) < d) ++f.shift;
    f.mul = (unsigned)(((1ull << 32) * ((1ull << f.shift) - d)) / d + 1);
    return f;
  }
  __host__ __device__ int div(int t) const {
    const unsigned u = (unsigned)t;
    return (int)(((unsigned)(((unsigned long long)mul * u) >> 32) + u) >> shift);
  }
};

inline bool tile_supported(int elem_bytes, int ns, int np, int code) {
  return code == kTileWave ? wave_variant_supported(elem_bytes, ns, np) : cpt_supported(elem_bytes, ns, code);
}
// the wave variant wherever it exists (three states: 1.3-2.1x faster than
// the workgroup variant on 128x128 and 256x256 batches of 3-16 members)
inline int tile_default(int elem_bytes, int ns, int np) {
  return wave_variant_supported(elem_bytes, ns, np) ? kTileWave : cpt_default(elem_bytes, ns);
}

// Arguments of the fused RK-stage kernel (passed by value).
struct StageArgs {
  const void* v;         // stage input, packed [B][N+1][nc][nq][np]
  const void* y;         // RK4 base state (nullptr: treated as zero)
  void* out;             // y + coef * L v
  double* partials;      // [B][npartials] level-0 trace partials of one sample, or nullptr
  const void* twiddle2;  // [n1][n2+1] complex exp(+2 pi i (n2 k1 mod np)/np), state precision, of the variant's plan
  const void* dtab;      // [ns][nq][np]: (U_j(q+r/2) - U_j(q-r/2)) / (2 hbar np), 0 at Nyquist
  const void* gtab;      // [npair][nq][np]: (U_j(q+r/2) - U_k(q-r/2)) / (hbar np), j < k
  const void* ctab;      // [npair][2][nq][np]: U_jl(q + r/2), U_jl(q - r/2) / (hbar np), pair j < l
                         // (q-dependent couplings in the workgroup variant)
  const void* mtab;      // wave variant: [kWaveTables][nq][n1][n2] = dtab 0 + dtab 1, dtab 0 - dtab 1, gtab,
                         // U_01(q + r/2), U_01(q - r/2) (both / (hbar np)), entry (k1, k2) at m = k1 + n1 k2;
                         // three states: [kWaveTables3][nq][n1][n2] = the same sum and difference, dtab 2, gtab 0..2
  const double* bath;    // [B][kBathStride]: r0/m (= zeta), gamma, c0, c_delta, beta per member
  const void* psym;      // [2][np]: DFT symbols of D_p2 and D_p D_p, divided by np
  const void* closure;   // wave variant: learned W^(N+1) [B][4][nq][np] (one level per member), or nullptr
  // per-member depths (nullptr: every member has `depth`): member b has
  // levels mlev[b] .. mlev[b + 1] - 1 of a row numbering over all members,
  // and lev_member[row] is the member of a row.  mfirst: the member (in
  // that numbering) of this launch's member 0.
  const int* mlev;
  const int* lev_member;
  int mfirst;
  int qcoup;  // 1: q-dependent coupling through the r-space multiply (wave variant, two states)
  int nq;
  int depth;
  int ntiles;
  int batch;
  int nblocks_padded;       // grid size: ntiles * (depth+1) * batch rounded up to a multiple of 8
  int stream_out;           // wave variant: 1 = non-temporal output stores (the state arrays are well
                            // past the memory-side cache)
  WaveShape shape;          // wave variant
  int npartials;            // trace partials per member (wave variant: one per column)
  FixedDiv by_levels, by_tiles;  // division by depth + 1 and by ntiles
  double inv_60dq, inv_12dp;     // 1 / (60 dq), 1 / (12 dp)
  long long member_stride;  // elements per member
  long long level_stride;   // elements per level
  long long comp_stride;    // elements per packed component (nq * np)
  double coef;
  double dq, dp, p0;
  double inv_mass;
  double coup[QHFPE_MAX_STATES][QHFPE_MAX_STATES];     // off-diagonal couplings / hbar
  double mu[QHFPE_MAX_STATES][QHFPE_MAX_STATES];
};

// Learned terminator (closure.hip): a linear 13x13 convolution over (q, p)
// from 8 input channels (the packed components of level N and the same times
// p) to the 4 packed components of level N + 1, trained as three 5x5 layers
// with kClosureHidden channels.
constexpr int kClosureHalf = 6;
constexpr int kClosureIn = 8;
constexpr int kClosureOut = 4;
constexpr int kClosureHidden = 32;
constexpr int kClosureKernelElems = 13 * 13 * kClosureIn * kClosureOut;   // K[13][13][8][4]
constexpr int kClosureStatsA = 25 * 25 * kClosureIn * kClosureIn;         // A[25][25][8][8]
constexpr int kClosureStatsC = 13 * 13 * kClosureIn * kClosureOut;        // C[13][13][8][4]
constexpr int kClosureStatsSize = kClosureStatsA + kClosureStatsC + 1;    // + yy
constexpr int kClosureWeightElems = 16 * 7 * 16 * 16;                     // BF16 MFMA B layout
// Training state (floats): the three layers, the layers after the running
// iteration (the two buffers swap from iteration to iteration), Adam moments,
// the 9x9 product of the first two layers and its gradient, the composite
// kernel and its gradient, and per-entry loss terms (doubles).
struct ClosureTrainLayout {
  static constexpr int w1 = 0, n1 = 25 * kClosureIn * kClosureHidden;
  static constexpr int w2 = w1 + n1, n2 = 25 * kClosureHidden * kClosureHidden;
  static constexpr int w3 = w2 + n2, n3 = 25 * kClosureHidden * kClosureOut;
  static constexpr int nparam = n1 + n2 + n3;
  static constexpr int g1 = nparam, g2 = g1 + n1, g3 = g2 + n2;
  static constexpr int m = 2 * nparam, v = 3 * nparam;
  static constexpr int w12 = 4 * nparam, n12 = 81 * kClosureIn * kClosureHidden;
  static constexpr int g12 = w12 + n12;
  static constexpr int k = g12 + n12;
  static constexpr int gk = k + kClosureKernelElems;
  static constexpr int terms = gk + kClosureKernelElems;  // kClosureKernelElems doubles
  static constexpr int loss = terms + 2 * kClosureKernelElems;  // one double
  static constexpr int total = loss + 2;
};
static_assert(ClosureTrainLayout::terms % 2 == 0 && ClosureTrainLayout::loss % 2 == 0, "doubles stay aligned");

hipError_t launch_closure_weights(const float* K, unsigned short* wb, hipStream_t s);
hipError_t launch_closure_apply(int precision, int np, const void* v, int level, long long member_stride,
                                long long level_stride, long long comp_stride, int nq, int batch, double p0,
                                double dp, const unsigned short* wb, void* out, long long out_stride, hipStream_t s);
// scratch: at least closure_stats_scratch_bytes() of device memory for the
// partial sums; more lets more workgroups take part
size_t closure_stats_scratch_bytes();
hipError_t launch_closure_stats(int precision, int np, const void* v, int level, long long member_stride,
                                long long level_stride, long long comp_stride, int nq, int batch, double p0,
                                double dp, double* scratch, size_t scratch_bytes, double* stats, hipStream_t s);
hipError_t launch_closure_train_step(const double* stats, const float* prior, double ridge, float* state, int from,
                                     int to, int t, float lr, hipStream_t s);
hipError_t launch_closure_compose(const double* stats, float* state, double* loss, hipStream_t s);
hipError_t launch_closure_loss(const double* stats, const float* K, float* g, double* terms, double* loss,
                               hipStream_t s);

// Host launchers (one translation unit per precision and state count).
hipError_t launch_stage_f64_ns2(int np, int cpt, const StageArgs& a, int nblocks, hipStream_t s);
hipError_t launch_stage_f64_ns3(int np, int cpt, const StageArgs& a, int nblocks, hipStream_t s);
hipError_t launch_stage_f32_ns2(int np, int cpt, const StageArgs& a, int nblocks, hipStream_t s);
hipError_t launch_stage_f32_ns3(int np, int cpt, const StageArgs& a, int nblocks, hipStream_t s);
hipError_t launch_stage_wave_f64_ns2(int np, const StageArgs& a, int nblocks, hipStream_t s);
hipError_t launch_stage_wave_f64_ns3(int np, const StageArgs& a, int nblocks, hipStream_t s);
hipError_t launch_stage_wave_f32_ns2(int np, const StageArgs& a, int nblocks, hipStream_t s);
hipError_t launch_stage_wave_f32_ns3(int np, const StageArgs& a, int nblocks, hipStream_t s);

// Pointwise and reduction kernels (aux_kernels.hip).
struct DipoleMu {
  double m[QHFPE_MAX_STATES][QHFPE_MAX_STATES];
};

struct GridDesc {
  int ns, nq, np, levels, batch, precision;
  long long member_stride, level_stride, comp_stride;
};

hipError_t launch_pack(const GridDesc& g, const double* canon, int phase, void* packed,
                       int member_offset, int nmembers, double* red, int* nred_blocks,
                       hipStream_t s);
hipError_t launch_unpack(const GridDesc& g, const void* packed, int phase, double* canon,
                         int member_offset, int nmembers, hipStream_t s);
hipError_t launch_dipole(const GridDesc& g, void* packed, const double mu[3][3], hipStream_t s);
hipError_t launch_thermal(const GridDesc& g, void* packed, double q0, double dq, double p0,
                          double dp, const double* bath, double omega, double mass, double hbar,
                          const double* noise, hipStream_t s);
hipError_t launch_trace_partials(const GridDesc& g, const void* packed, const double mu[3][3],
                                 int tq, int ntiles, double* partials, hipStream_t s);
// partials of member b's sample j: partials + j slot_stride + b ntiles
hipError_t launch_finalize(int batch, int ntiles, int nslots, const double* partials, long long slot_stride,
                           double scale, int phase, double* resp, long long resp_stride,
                           long long resp_offset, int* flag, hipStream_t s);
hipError_t launch_clear_flag(int* flag, hipStream_t s);
// device-to-device copy of `bytes` (dst and src 16-byte aligned) by a
// streaming kernel: no memcpy or memset node when captured into a graph
hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t s);
hipError_t launch_norm_partials(const GridDesc& g, const void* packed, double* red,
                                int* nblocks_per_member, hipStream_t s);
hipError_t launch_spectrum_abs(const double* series, long long n, double dt, const double* omega,
                               int n_omega, double* out, hipStream_t s);
// The fixed device scratch of qhfpe_spectrum_corr_noalloc: kScratchDoubles
// doubles per device; scratch_pointer() returns the current device's address.
constexpr size_t kScratchDoubles = size_t(1) << 17;  // 1 MiB
constexpr int kMaxDevices = 64;
hipError_t scratch_pointer(double** out);
hipError_t launch_spectrum_corr(const double* r3, int n1, int n3, double dt1, double dt3,
                                const double* w1, int nw1, const double* w3, int nw3,
                                double* work, double* out, hipStream_t s);

}  // namespace qhfpe
