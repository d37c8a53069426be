// Fused RK4 stage, wave-independent variant:  out = y + coef * L v  with the
// same operator as stage_kernel.hpp (Eq. (heom) of Ikeda & Tanimura (2017)
// with one Drude exponential and V(q) = q, closed by Eq. (GMFP); potential
// term of Eq. (quantum-liouvillian) through the DFT along p; Sec. III
// discretisation), for two and three electronic states and np = 32 .. 256.
//
// One wave owns a whole task: neighbouring q columns of one level of one batch
// member, all packed components.  A column's p nodes lie on L = 16, 32 or 64
// lanes, K consecutive nodes each; the wave holds G = 64 / L groups of lanes
// with C columns each (TQ = G C columns per task).  The waves of a workgroup
// share only the twiddle and symbol tables (loaded once behind the single
// workgroup barrier); every later step orders its LDS accesses within the
// wave, so a wave waiting for memory never stalls another.
//
//  - kinetic -(p/m) D_q: 5th-order upwind over a (C + 6)-column q window;
//  - D_p of the level field g: the stencil neighbours p +- 1, +- 2 of a
//    lane's nodes are its own or the neighbouring lanes' (rotations within the
//    L lanes; the p grid is periodic and one column fills them);
//  - potential term: complex np-point transforms (the two real diagonals of a
//    column packed into one, each coherence in another, and with three states
//    the third diagonals), two-pass FFT np = N1 N2 in
//    rounds of 64 items, r-space multiply in place (a round holds whole
//    transforms, and its lanes read their own and partner rows before any
//    of them writes), inverse transform;
//  - constant diabatic coupling: pointwise commutator in p; a q-dependent
//    coupling U_01(q) (two states) instead enters the r-space multiply (QC
//    instantiation), where it mixes the packed-diagonal and coherence
//    transforms of a column.
//
// What bounds it: a small launch (each wave on a SIMD of its own) by one
// wave's chain of launch, loads and FFT rounds, a large one by how well the
// waves' load and transform phases overlap (no unit is saturated: 1024 members
// of 128 x 128 x 7 levels in FP32 take 1.18 ms, of which VALU issue is 0.65, 1751
// instructions a wave, and their 4.9 GB at the copy rate 0.89).  wave_shape (qhfpe_internal.hpp) holds the
// rule and its measurements.  Against one fixed shape at 128 and 256 and the
// workgroup variant elsewhere (us per stage, FP64): 48 x 48 x 4 levels, one
// member 11.4 -> 5.5; 128 x 128 x 7 one member 10.9 -> 6.5; 96 x 96 x 7 four members
// 13.0 -> 10.5; 192 x 192 x 9 sixteen members 171 -> 120; three states 64 x 64 x 3
// sixty members 82.5 -> 36.6; 256 x 256 x 9 two members 25.5 -> 21.9.
//
// Every column is computed by the same operations in the same order whatever
// C, PF and the workgroup shape are (contraction is off, the fused
// operations are written out, and the trace partials are one per column), so a
// launch may take the shape that suits its size and the results stay the same
// bit for bit.
#pragma once

#include "device_common.hpp"
#include "qhfpe_internal.hpp"
#include "stage_kernel.hpp"

namespace qhfpe {

template <int NS_, int NP_, int C_, int WPB_>
struct WavePlan {
  static constexpr int NS = NS_, NP = NP_, C = C_;
  static constexpr int N1 = wave_n1(NP), N2 = NP / N1;
  static constexpr int K = wave_nodes(NP);     // p nodes per lane
  static constexpr int L = NP / K;             // lanes per column
  static constexpr int G = 64 / L;             // lane groups
  static constexpr int TQ = G * C;             // q columns per task
  static constexpr int NC = NS * NS;           // packed components
  static constexpr int NPAIR = NS * (NS - 1) / 2;
  // complex transforms per task: f < TQ the diagonal pair (0, 1) of column f;
  // then each coherence pair's of every column; with three states then the
  // W22s: of columns 2 h (real part) and 2 h + 1 (imaginary) where the wave
  // holds several lane groups, else of one column each with a zero imaginary
  // part (so that a column's rounding does not depend on C; the count of
  // rounds is the same)
  static constexpr int F22 = TQ * (1 + NPAIR);
  static constexpr bool kPair22 = G > 1;
  static constexpr int NF = F22 + (NS == 3 ? (kPair22 ? TQ / 2 : TQ) : 0);
  static constexpr int P1 = NF * N2, P2 = NF * N1;  // items of the strided and the contiguous passes
  static constexpr int R1 = (P1 + 63) / 64, R2 = (P2 + 63) / 64;
  static constexpr int WPB = WPB_;  // waves per workgroup
  static constexpr int NT = 64 * WPB;
  // LDS: one column of complex values per transform, one element of padding
  // per N2 block.  The column stride keeps the lanes of the strided passes,
  // which hold neighbouring columns, on different banks (128: eight lanes a
  // column, so a stride of 24 mod 32).
  static constexpr int LDP = NP == 128 ? 152 : NP + NP / N2;
  // the transform that holds packed component comp of task column i, and
  // whether as its real (0) or imaginary (1) part
  __host__ __device__ static constexpr int transform(int i, int comp) {
    if (comp < 2) return i;
    if (NS == 3 && comp == 2) return F22 + (kPair22 ? i / 2 : i);
    return TQ * (1 + (comp - NS) / 2) + i;
  }
  __host__ __device__ static constexpr int part(int i, int comp) {
    if (comp < 2) return comp;
    if (NS == 3 && comp == 2) return kPair22 ? i % 2 : 0;
    return (comp - NS) % 2;
  }
  // W22 does not share its transform with another component of its column
  __host__ __device__ static constexpr bool alone(int comp) { return NS == 3 && comp == 2; }
  static_assert(K * L == NP && (L == 16 || L == 32 || L == 64) && 64 % N1 == 0 && N1 * N2 == NP && N2 % 2 == 0, "wave plan");
};

// complex values in LDS: one 8- or 16-byte access each
template <typename T>
using lds_cx = T __attribute__((ext_vector_type(2)));

// 16-point DFTs shared by four lanes each, for launches whose waves have idle
// lanes in the FFT rounds (one lane alone takes 16 points in a chain of about
// 160 operations).  Item i's points lie at pts(i)[stride k]; sub-lane j of an
// item computes the j-th four-point DFT of either half of the 4 x 4
// factorisation, with the operations and constants of SmallDft<16> (the same
// bits), in two LDS round trips.  out(i, k, X_k) returns what is stored at
// position k.  A stage of 128 x 64 x 4 levels, one column a wave, takes 5.95 us
// instead of 6.95 (FP64), 128 x 128 x 7 6.1 instead of 6.6 (FP32).
template <int S, typename T, typename Pts, typename Out>
__device__ __forceinline__ void dft16_four_lanes(int lane, int items, int stride, Pts pts, Out out) {
#pragma clang fp contract(off)
  const int rounds = (4 * items + 63) / 64;  // (a constant once inlined)
  const int j = lane & 3;
  // w16^(j k1), k1 = 1..3
  T wc[3], ws[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int e1 = 3 * (k + 1), e2 = 6 * (k + 1), e3 = 9 * (k + 1);
    wc[k] = j == 0 ? T(1) : (j == 1 ? T(kCos48[e1]) : (j == 2 ? T(kCos48[e2]) : T(kCos48[e3])));
    ws[k] = j == 0 ? T(0) : (j == 1 ? T(S * kSin48[e1]) : (j == 2 ? T(S * kSin48[e2]) : T(S * kSin48[e3])));
  }
#pragma unroll
  for (int t = 0; t < rounds; ++t) {
    const int item = (lane >> 2) + 16 * t;
    if (4 * items % 64 == 0 || t + 1 < rounds || item < items) {
      lds_cx<T>* const z = pts(item) + j * stride;
      cx<T> x[4];
#pragma unroll
      for (int n1 = 0; n1 < 4; ++n1) x[n1] = {z[4 * n1 * stride][0], z[4 * n1 * stride][1]};
      SmallDft<4, S, T>::run(x);
#pragma unroll
      for (int k1 = 1; k1 < 4; ++k1) x[k1] = cmul(x[k1], cx<T>{wc[k1 - 1], ws[k1 - 1]});
#pragma unroll
      for (int k1 = 0; k1 < 4; ++k1) z[4 * k1 * stride] = lds_cx<T>{x[k1].re, x[k1].im};
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int t = 0; t < rounds; ++t) {
    const int item = (lane >> 2) + 16 * t;
    const bool on = 4 * items % 64 == 0 || t + 1 < rounds || item < items;
    cx<T> x[4];
    if (on) {
      const lds_cx<T>* const z = pts(item) + 4 * j * stride;
#pragma unroll
      for (int n2 = 0; n2 < 4; ++n2) x[n2] = {z[n2 * stride][0], z[n2 * stride][1]};
      SmallDft<4, S, T>::run(x);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) x[k2] = out(item, j + 4 * k2, x[k2]);
    }
    wave_lds_sync();  // an item's lanes share a round: all have read
    if (on) {
      lds_cx<T>* const z = pts(item) + j * stride;
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) z[4 * k2 * stride] = lds_cx<T>{x[k2].re, x[k2].im};
    }
  }
}

// C: columns per lane group.  PF: components whose loads are in flight (each
// holds its window and neighbour levels in registers): component c + PF
// takes c's registers once c is done; kStaggered: one in flight at the start,
// then c + 1's window is issued after c's kinetic term and its neighbour
// levels after c's.  OCC: waves per SIMD the register allocation
// aims at.  QC: q-dependent diabatic coupling
// U_01(q), applied in the r-space multiply.  NTS: non-temporal output stores
// (StageArgs::stream_out).  WPB: waves per workgroup (StageArgs::shape).  MIX:
// members of their own depths (StageArgs::mlev).
template <typename T, int NS, int NP, int C, int PF, int OCC, bool QC, bool NTS, int WPB, bool MIX>
__global__ void __launch_bounds__(64 * WPB, OCC) stage_wave_kernel(StageArgs a) {
#pragma clang fp contract(off)
  using W = WavePlan<NS, NP, C, WPB>;
  constexpr int N1 = W::N1, N2 = W::N2, K = W::K, L = W::L, TQ = W::TQ, NC = W::NC, NF = W::NF;
  constexpr int R1 = W::R1, R2 = W::R2, P1 = W::P1, P2 = W::P2, LDP = W::LDP;
  static_assert(!QC || NS == 2, "q-dependent couplings: two states");
  constexpr bool kStag = PF == kStaggered;
  constexpr bool kAll = PF >= NC;  // every load in flight at once
  constexpr int SL = kStag ? 2 : (kAll ? NC : PF);  // register slots for components
  auto pad = [](int x) { return x + x / N2; };  // padded position of p node x in a column
  __shared__ lds_cx<T> sbuf[WPB][NF * LDP];    // per wave: v tile, transformed in place
  __shared__ lds_cx<T> stw[N1 * (N2 + 1)];     // w^(n2 k1), row k1 padded to N2 + 1
  constexpr int NSYM = NP / 2 + 1;
  __shared__ T ssym[2 * NSYM];  // DFT symbols of D_p2 and D_p D_p (scaled by 1/np; even in m)

  // A small launch starts with the arguments' scalar loads: left to itself the
  // compiler fetches them where they are used, five round trips in a row before
  // the first state load.  Fetched together (with the short address arithmetic
  // below) a stage of 128 x 64 x 4 levels takes 5.6 us instead of 5.95 (FP64),
  // 48 x 48 x 4 5.5 instead of 5.9, two members of 256 x 256 x 9 24.5 instead of
  // 25.2.  The largest launches (four waves a workgroup) lose half a percent.
  if constexpr (!MIX && WPB <= 2) {
    asm volatile("" ::"s"(a.v), "s"(a.y), "s"(a.out), "s"(a.mtab), "s"(a.bath), "s"(a.twiddle2), "s"(a.psym), "s"(a.closure),
                 "s"(a.nblocks_padded), "s"(a.nq), "s"(a.depth), "s"(a.ntiles), "s"(a.batch));
    asm volatile("" ::"s"(a.by_levels.mul), "s"(a.by_levels.shift), "s"(a.by_tiles.mul), "s"(a.by_tiles.shift),
                 "s"(a.member_stride), "s"(a.level_stride), "s"(a.comp_stride));
  }
  const int tid = threadIdx.x;
  // the wave index is uniform across the wave; saying so keeps every
  // quantity derived from it (task, level, member, buffer descriptors) in
  // scalar registers instead of per-lane loops over descriptor values
  const int lane = tid & 63, wid = WPB == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nq = a.nq;
  const int ntasks = stage_units<MIX>(a);
  // levels fastest, as in stage_kernel: the tasks of all levels of one
  // column group run together and share their level neighbours through L2
  const int task_id = xcd_logical_block(blockIdx.x, a.nblocks_padded) * WPB + wid;
  // a wave past the last task still meets its workgroup at the table
  // barrier below; it takes task 0's indices and ends after the barrier
  const bool active = task_id < ntasks;
  if (WPB == 1 && !active) return;
  const int task = active ? task_id : 0;
  const UnitPos pos = unit_pos<MIX, true>(a, task);
  const int n = pos.n, tile = pos.tile, b = pos.b;
  const int grp = L == 64 ? 0 : lane / L, lig = L == 64 ? lane : lane % L;
  const int c0l = C * grp;            // this lane's first task column
  const int q0 = TQ * tile;           // the task's first q column
  lds_cx<T>* const s = sbuf[wid];
  // element of component comp of task column i at p node x
  auto elem = [&](int i, int comp, int x) -> T& {
    return reinterpret_cast<T*>(s)[2 * (W::transform(i, comp) * LDP + x + x / N2) + W::part(i, comp)];
  };

  constexpr unsigned ES = sizeof(T);
  const unsigned level_bytes = (unsigned)(a.level_stride * ES);
  const unsigned cbytes = (unsigned)(a.comp_stride * ES);
  const unsigned long long at_member = (unsigned long long)a.member_stride * (unsigned)b * ES;
  const unsigned long long at_level = at_member + (unsigned long long)level_bytes * (unsigned)n;
  auto at = [](const void* base, unsigned long long bytes) { return static_cast<const char*>(base) + bytes; };
  // Loads past a descriptor's size return zero.  That supplies the zero
  // ghost columns beyond the q edges (their offsets are set past every
  // level), v^(n+1) at n = N, v^(n-1) at n = 0 and a missing y.
  const bool has_up = n < pos.depth, has_dn = n >= 1;
  // learned terminator: at n = N the level above is the closure's W^(N+1)
  const bool clos = NS == 2 && a.closure != nullptr && !has_up;
  const rsrc_t rn = make_rsrc(at(a.v, at_level), level_bytes);
  const rsrc_t ru = make_rsrc(at(clos ? a.closure : a.v, clos ? (unsigned long long)level_bytes * (unsigned)b
                                                              : at_level + level_bytes),
                              has_up || clos ? level_bytes : 0u);
  const rsrc_t rd = make_rsrc(at(a.v, at_level - (has_dn ? level_bytes : 0u)), has_dn ? level_bytes : 0u);
  const bool has_y = a.y != nullptr;
  const rsrc_t ry = make_rsrc(at(a.y, has_y ? at_level : 0ull), has_y ? level_bytes : 0u);

  // (the bath constants' scalar loads are issued here, long before their use)
  const double* bath = a.bath + kBathStride * b;
  const double bath_zeta = bath[0], bath_gamma = bath[1], bath_c0 = bath[2], bath_cdel = bath[3];

  const int a0 = K * lig;  // first p node of this lane
  // byte offsets of the lane's q columns -3 .. C+2 at its first node; columns
  // outside the grid point past the end of every level (read as 0)
  constexpr unsigned kGhost = 0x7fffff00u;
  unsigned qo[C + 6];
#pragma unroll
  for (int t = 0; t < C + 6; ++t) {
    const int q = q0 + c0l + t - 3;
    qo[t] = (q >= 0 && q < nq) ? ((unsigned)q * NP + a0) * ES : kGhost;
  }

  // ---- loads -------------------------------------------------------------
  // v^(n) at the task columns is the middle of the kinetic window, so it is
  // loaded once
  T loc[C][NC][K];     // all terms of L v except the potential's
  T lw[SL][2][C][K];   // v^(n+1), v^(n-1) at the task columns
  T kw[SL][C + 6][K];  // kinetic window
  T ky[C][NC][K];      // y at the task columns
  auto issue_window = [&](int comp) {
    const unsigned so = comp * cbytes;
    const int sl = comp % SL;
#pragma unroll
    for (int t = 0; t < C + 6; ++t) buf_load_n<K>(rn, qo[t], so, kw[sl][t]);
  };
  auto issue_level = [&](int comp) {
    const unsigned so = comp * cbytes;
    const int sl = comp % SL;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      buf_load_n<K>(ru, qo[i + 3], so, lw[sl][0][i]);
      buf_load_n<K>(rd, qo[i + 3], so, lw[sl][1][i]);
    }
  };
  auto issue = [&](int comp) {
    issue_window(comp);
    issue_level(comp);
  };
  // y enters only the last line (one rounding at its magnitude).  Its loads are
  // issued before the last FFT pass, which hides them and spreads the wave's
  // loads over its time; a wave of a small launch, which has registers to
  // spare, issues them and its multipliers' before the first FFT pass.
  auto issue_y = [&]() {
#pragma unroll
    for (int comp = 0; comp < NC; ++comp)
#pragma unroll
      for (int i = 0; i < C; ++i) buf_load_n<K>(ry, qo[i + 3], comp * cbytes, ky[i][comp]);
  };
  // r-space multipliers of this lane's items (host-permuted so that the N2
  // values of row k1 are contiguous): Y = -i [ s Z[m] + d conj(Z[-m]) ] + e Z
  // with s, d the sum and difference of the packed diagonals' tables, or s = g
  // and d = 0 (an offset past the table) for a coherence
  const unsigned tbytes = (unsigned)((long long)nq * NP * ES);
  constexpr int kPlanes = NS == 3 ? kWaveTables3 : kWaveTables;
  const rsrc_t rt = make_rsrc(a.mtab, (unsigned)kPlanes * tbytes);
  constexpr int MV = N2 % 4 == 0 ? 4 : 2;
  // rounds of one kind only: the kind is then known at compile time (after
  // unrolling) and a coherence round needs no partner rows
  constexpr bool kUniform = (TQ * N1) % 64 == 0;
  auto coherence_round = [&](int t) { return kUniform && 64 * t >= TQ * N1 && 64 * t < W::F22 * N1; };
  auto has_w22 = [&](int t) { return NS == 3 && 64 * t + 63 >= W::F22 * N1; };
  auto load_mul = [&](int t, T* mS, T* mD) {
    const int item = min(lane + 64 * t, P2 - 1);
    const int f = item / N1, k1 = item % N1;
    const bool w22 = has_w22(t) && f >= W::F22;
    const int kind = w22 ? 0 : f / TQ;  // 0: packed diagonals, 1 + pair: coherences
    const int col = w22 ? (W::kPair22 ? 2 : 1) * (f - W::F22) : f % TQ;
    const unsigned row = (unsigned)min(q0 + col, nq - 1) * NP + (unsigned)k1 * N2;
    // planes: two states s, d, g (then U_01 +-); three states s, d, U_22's, g of the pairs
    const unsigned pa = w22 ? 2u : (kind == 0 ? 0u : (unsigned)(NS == 3 ? 2 + kind : 2));
    const unsigned oa = pa * tbytes + row * ES;
    unsigned od = kind == 0 ? tbytes + row * ES : 0xfffff000u;  // (past the planes, which take up to 2.7 GB)
    if (has_w22(t) && w22) {
      // W22 of two columns: the tables of either; s and d are formed below
      const int colb = W::kPair22 ? col + 1 : col;
      od = 2 * tbytes + ((unsigned)min(q0 + colb, nq - 1) * NP + (unsigned)k1 * N2) * ES;
    }
#pragma unroll
    for (int k2 = 0; k2 < N2; k2 += MV) {
      buf_load_n<MV>(rt, oa + k2 * ES, 0, mS + k2);
      if (!coherence_round(t)) buf_load_n<MV>(rt, od + k2 * ES, 0, mD + k2);
    }
  };
  constexpr bool kHeld = WPB == 1 || QC;  // every round's multipliers in registers at once
  T mulS[kHeld ? R2 : 2][N2], mulD[kHeld ? R2 : 2][N2];

  // The twiddle and symbol tables go to LDS behind the workgroup's only
  // barrier.  Their loads are issued first and the first components' loads
  // right after them, so that the wait for the tables (loads complete in
  // issue order) does not wait for the components and the components'
  // latency overlaps the table stores and the barrier.
  {
    constexpr int NTW = N1 * (N2 + 1), NSY = 2 * NSYM;
    constexpr int RTW = (NTW + W::NT - 1) / W::NT, RSY = (NSY + W::NT - 1) / W::NT;
    T twr[RTW][2], syr[RSY];  // (plain scalars: an array of cx<T> went to scratch)
    // (lanes past a table's end load its last entry and store nothing, so
    // that the loads need no branch)
#pragma unroll
    for (int r = 0; r < RTW; ++r) {
      const T* const t = static_cast<const T*>(a.twiddle2) + 2 * min(tid + r * W::NT, NTW - 1);
      twr[r][0] = t[0];
      twr[r][1] = t[1];
    }
#pragma unroll
    for (int r = 0; r < RSY; ++r) {
      const int j = min(tid + r * W::NT, NSY - 1);
      syr[r] = static_cast<const T*>(a.psym)[j < NSYM ? j : j + NP - NSYM];
    }
    __builtin_amdgcn_sched_barrier(0);
    // (an inactive wave loads task 0's data too: in bounds, and no branch)
#pragma unroll
    for (int comp = 0; comp < (kStag ? 1 : SL); ++comp) issue(comp);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < RTW; ++r) {
      const int j = tid + r * W::NT;
      if (j < NTW) stw[j] = lds_cx<T>{twr[r][0], twr[r][1]};
    }
#pragma unroll
    for (int r = 0; r < RSY; ++r) {
      const int j = tid + r * W::NT;
      if (j < NSY) ssym[j] = syr[r];
    }
    __syncthreads();  // the only workgroup barrier
  }
  if (!active) return;

  // ---- constants of this lane --------------------------------------------
  const T zeta = T(bath_zeta), c0 = T(bath_c0), cdel = T(bath_cdel);
  const T ng = T(n * bath_gamma);
  const T coef = T(a.coef);
  // the terminator level differentiates zeta p v^(N) in place of v^(N+1)
  // (Eq. (GMFP)), unless a learned closure supplies W^(N+1)
  const T zterm = (has_up || clos) ? T(0) : zeta;
  const T ngc0 = ng * c0, dpinv = T(a.inv_12dp);
  T kscale[K], zp[K], nzp[K];
  bool pos_p[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const T p = T(fma_((double)(a0 + j), a.dp, a.p0));
    pos_p[j] = p >= T(0);
    kscale[j] = -(p * T(a.inv_mass)) * T(a.inv_60dq);
    zp[j] = zterm * p;
    nzp[j] = (ng * zeta) * p;
  }
  // upwind coefficients (x60) on q offsets -3..3 for the sign of p at this
  // lane's first node; nodes of the other sign (only where p = 0 falls
  // inside a lane) are redone below
  T kc[7];
#pragma unroll
  for (int o = -3; o <= 3; ++o) {
    const double cp = (o <= 2) ? kUpwind[o + 3] : 0.0;
    const double cn = (o >= -2) ? -kUpwind[3 - o] : 0.0;
    kc[o + 3] = T(pos_p[0] ? cp : cn);
  }
  const bool any_mixed = K > 1 && __any(pos_p[K - 1] != pos_p[0]);

  // ---- local terms, one component at a time ------------------------------
  // constant diabatic coupling -(i/hbar) [Delta, W] (pointwise in p).  Two
  // states: with d = Delta_01 / hbar it adds -2 d Im W01 to W00, +2 d Im W01
  // to W11, 0 to Re W01 and d (W00 - W11) to Im W01; it is applied with the
  // last component, reading W00 and W11 back from this lane's own LDS entries
  const bool has_coup = NS == 2 && a.coup[0][1] != 0.0;
  const T dcoup = T(a.coup[0][1]);
#pragma unroll
  for (int comp = 0; comp < NC; ++comp) {
    const int sl = comp % SL;
    // kinetic term at the lane's nodes of every column
    T kin[C][K];
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int j = 0; j < K; ++j) {
        T k = kc[0] * kw[sl][i][j];
#pragma unroll
        for (int o = 1; o < 7; ++o) k = fma_(kc[o], kw[sl][i + o][j], k);
        if (K > 1 && any_mixed && pos_p[j] != pos_p[0]) {
          // where p = 0 falls inside a lane, its nodes of the other sign
          // take the mirrored stencil
          k = -kc[6] * kw[sl][i][j];
#pragma unroll
          for (int o = 1; o < 7; ++o) k = fma_(-kc[6 - o], kw[sl][i + o][j], k);
        }
        kin[i][j] = kscale[j] * k;
        if constexpr (!kAll) asm volatile("" : "+v"(kin[i][j]));
      }
    if constexpr (!kAll) __builtin_amdgcn_sched_barrier(0);
    if constexpr (kStag) {
      if (comp + 1 < NC) issue_window(comp + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    // level field and level terms
#pragma unroll
    for (int i = 0; i < C; ++i) {
      T g[K], lev[K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const T w0 = kw[sl][i + 3][j];
        // field differentiated once along p:
        //   n < N: v^(n+1) + n gamma c0 v^(n-1);  n = N: zeta p v^(N) + N gamma c0 v^(N-1)
        // (the absent neighbour levels read as zero; n gamma = 0 at n = 0)
        g[j] = fma_(ngc0, lw[sl][1][i][j], fma_(zp[j], w0, lw[sl][0][i][j]));
        lev[j] = fma_(nzp[j], lw[sl][1][i][j], -(ng * w0));
        elem(c0l + i, comp, a0 + j) = w0;
        if (NS == 3 && !W::kPair22 && comp == 2)
          reinterpret_cast<T*>(s)[2 * ((W::F22 + c0l + i) * LDP + pad(a0 + j)) + 1] = T(0);
      }
      // D_p g: nodes a0-2, a0-1 come from the previous lane, a0+K, a0+K+1
      // from the next one (periodic in p: a column fills the lane group)
      T e[K + 4];
      if constexpr (K == 1) {
        e[1] = lane_prev<L>(g[0]);
        e[0] = lane_prev<L>(e[1]);
        e[K + 2] = lane_next<L>(g[0]);
        e[K + 3] = lane_next<L>(e[K + 2]);
      } else {
        e[0] = lane_prev<L>(g[K - 2]);
        e[1] = lane_prev<L>(g[K - 1]);
        e[K + 2] = lane_next<L>(g[0]);
        e[K + 3] = lane_next<L>(g[1]);
      }
#pragma unroll
      for (int j = 0; j < K; ++j) e[j + 2] = g[j];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const T d = fma_(T(8), e[j + 3] - e[j + 1], e[j] - e[j + 4]);
        loc[i][comp][j] = fma_(dpinv, d, kin[i][j] + lev[j]);
        if (NS == 2 && comp == NC - 1 && has_coup) {
          const T w3 = kw[sl][i + 3][j];  // Im W01
          const lds_cx<T> h = s[(c0l + i) * LDP + pad(a0 + j)];  // W00, W11
          loc[i][0][j] = fma_(T(-2) * dcoup, w3, loc[i][0][j]);
          loc[i][1][j] = fma_(T(2) * dcoup, w3, loc[i][1][j]);
          loc[i][NC - 1][j] = fma_(dcoup, h[0] - h[1], loc[i][NC - 1][j]);
        }
        if constexpr (!kAll) asm volatile("" : "+v"(loc[i][comp][j]));
      }
    }
    if constexpr (!kAll) {
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (kStag) {
        if (comp + 1 < NC) issue_level(comp + 1);
      } else {
        if (comp + PF < NC) issue(comp + PF);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // three states: the couplings -(i/hbar) [Delta, W] from this lane's own LDS
  // entries of the nine components (each lane reads only what it wrote, so no
  // barrier is needed)
  if constexpr (NS == 3) {
    if (a.coup[0][1] != 0.0 || a.coup[0][2] != 0.0 || a.coup[1][2] != 0.0) {
      T cpl[3][3];
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int k = 0; k < 3; ++k) cpl[j][k] = T(a.coup[j][k]);
#pragma unroll
      for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < K; ++j) {
          T hv[NC], cm[NC];
#pragma unroll
          for (int comp = 0; comp < NC; ++comp) hv[comp] = elem(c0l + i, comp, a0 + j);
          commutator_mi<3, T>(cpl, hv, cm);
#pragma unroll
          for (int comp = 0; comp < NC; ++comp) loc[i][comp][j] += cm[comp];
        }
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < C; ++i)
#pragma unroll
    for (int comp = 0; comp < NC; ++comp)
#pragma unroll
      for (int j = 0; j < K; ++j) asm volatile("" : "+v"(loc[i][comp][j]));

  if constexpr (WPB == 1) {
    issue_y();
#pragma unroll
    for (int t = 0; t < R2; ++t) load_mul(t, mulS[t], mulD[t]);
  }

  // ---- potential term ----------------------------------------------------
  auto get = [](const lds_cx<T>& x) { return cx<T>{x[0], x[1]}; };
  auto put = [](cx<T> x) { return lds_cx<T>{x.re, x.im}; };

  // small launches share their 16-point DFTs between lanes
  // where the sub-items fit one round (np = 128).  With more rounds a lone member
  // of a small grid gains 4% but eight members lose 3 to 8% (192 and 256 points).
  constexpr bool kShare1 = WPB == 1 && NS == 2 && N1 == 16 && 4 * P1 <= 64;
  auto strided = [&](int item) { return s + item / N2 * LDP + item % N2; };

  // first forward pass: N1-point DFTs over stride N2, twiddle (item: f, n2)
  if constexpr (kShare1) {
    dft16_four_lanes<1, T>(lane, P1, N2 + 1, strided, [&](int item, int k1, cx<T> x) {
      return cmul(x, get(stw[k1 * (N2 + 1) + item % N2]));
    });
  }
#pragma unroll
  for (int t = 0; t < (kShare1 ? 0 : R1); ++t) {
    const int item = lane + 64 * t;
    if (P1 % 64 == 0 || t + 1 < R1 || item < P1) {
      const int n2 = item % N2;
      lds_cx<T>* const z = s + item / N2 * LDP + n2;
      cx<T> x[N1];
#pragma unroll
      for (int n1 = 0; n1 < N1; ++n1) x[n1] = get(z[(N2 + 1) * n1]);
      SmallDft<N1, 1, T>::run(x);
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) z[(N2 + 1) * k1] = put(cmul(x[k1], get(stw[k1 * (N2 + 1) + n2])));
    }
  }
  wave_lds_sync();

  // the multipliers: a round ahead, or all rounds' with a q-dependent coupling
  if constexpr (WPB > 1) {
#pragma unroll
    for (int t = 0; t < (QC ? R2 : 1); ++t) load_mul(t, mulS[t], mulD[t]);
  }
  // q-dependent coupling: U_01(q + r/2), U_01(q - r/2) of this lane's rows.
  // In FP32 they are loaded here with the other multipliers; in FP64 they
  // are loaded a few at a time inside the r-space loop, since holding all of
  // them through the forward passes would exceed the register budget.
  constexpr bool kQcEarly = QC && sizeof(T) == 4;
  auto qc_row = [&](int t) {
    const int item = min(lane + 64 * t, P2 - 1);
    const int f = item / N1, k1 = item % N1;
    return ((unsigned)min(q0 + f % TQ, nq - 1) * NP + (unsigned)k1 * N2) * ES;
  };
  T cP[kQcEarly ? R2 : 1][kQcEarly ? N2 : 1], cM[kQcEarly ? R2 : 1][kQcEarly ? N2 : 1];
  if constexpr (kQcEarly) {
#pragma unroll
    for (int t = 0; t < R2; ++t) {
      const unsigned row = qc_row(t);
#pragma unroll
      for (int k2 = 0; k2 < N2; k2 += MV) {
        buf_load_n<MV>(rt, 3u * tbytes + row + k2 * ES, 0, cP[t] + k2);
        buf_load_n<MV>(rt, 4u * tbytes + row + k2 * ES, 0, cM[t] + k2);
      }
    }
  }
  // second forward pass: contiguous N2-point DFTs of row k1 (item: f, k1).  Row
  // 0 also stores X[0] in its padding slot, so that the partner of index m
  // lies at pbase - k2 for every row
#pragma unroll
  for (int t = 0; t < R2; ++t) {
    const int item = lane + 64 * t;
    if (P2 % 64 == 0 || t + 1 < R2 || item < P2) {
      const int k1 = item % N1;
      lds_cx<T>* const z = s + item / N1 * LDP + (N2 + 1) * k1;
      cx<T> x[N2];
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) x[n2] = get(z[n2]);
      SmallDft<N2, 1, T>::run(x);
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) z[k2] = put(x[k2]);
      if (k1 == 0) z[N2] = put(x[0]);
    }
  }
  wave_lds_sync();

  // r-space multiplication (position k2 + (N2+1) k1 holds index
  // m = k1 + N1 k2) and the first inverse pass, round by round: a round holds
  // whole transforms, and its lanes read their own and partner rows before
  // any of them writes.  (A q-dependent coupling reads the column's other
  // transform, which may be in another round: there all rounds read before any
  // writes.)
  const T c0t = (has_up || clos) ? T(0) : c0;  // terminator level carries c0 D_p D_p
  cx<T> yk[QC ? R2 : 1][N2];
  auto write_back = [&](int t, cx<T>* y) {
    const int item = lane + 64 * t;
    if (P2 % 64 == 0 || t + 1 < R2 || item < P2) {
      const int k1 = item % N1;
      lds_cx<T>* const z = s + item / N1 * LDP + (N2 + 1) * k1;
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) z[n2] = put(cmulc(y[n2], get(stw[k1 * (N2 + 1) + n2])));
    }
  };
#pragma unroll
  for (int t = 0; t < R2; ++t) {
    if (!kHeld && t + 1 < R2) load_mul(t + 1, mulS[(t + 1) & 1], mulD[(t + 1) & 1]);
    T* const mS = mulS[kHeld ? t : t & 1];
    T* const mD = mulD[kHeld ? t : t & 1];
    cx<T>* const y = yk[QC ? t : 0];
    const int item = lane + 64 * t;
    if (P2 % 64 == 0 || t + 1 < R2 || item < P2) {
      const int k1 = item % N1;
      const int f = item / N1;
      const lds_cx<T>* const zf = s + f * LDP;
      const int rbase = (N2 + 1) * k1;
      const int pbase = (k1 == 0) ? N2 : (N2 - 1) + (N2 + 1) * (N1 - k1);
      // the other transform of the same column (q-dependent coupling only)
      const int kind = f / TQ;
      const lds_cx<T>* const zo = s + (f % TQ + TQ * (1 - kind)) * LDP;
      const T* const syp = ssym + k1;  // symbols at m = k1 + N1 k2, and at np - m for the upper half
      const T* const sym = ssym - k1;
      const T hk = kind ? T(0.5) : T(1);
      T qp[MV], qm[MV];  // FP64: the coupling values of a few k2
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2) {
        if constexpr (QC && !kQcEarly) {
          if (k2 % MV == 0) {
            __builtin_amdgcn_sched_barrier(0);
            buf_load_n<MV>(rt, 3u * tbytes + qc_row(t) + k2 * ES, 0, qp);
            buf_load_n<MV>(rt, 4u * tbytes + qc_row(t) + k2 * ES, 0, qm);
          }
        }
        const cx<T> z = get(zf[rbase + k2]);
        const T* const sy = k2 < N2 / 2 ? syp + N1 * k2 : sym + (NP - N1 * k2);
        const T e = fma_(cdel, sy[0], c0t * sy[NSYM]);
        if (coherence_round(t)) {
          y[k2] = {fma_(e, z.re, mS[k2] * z.im), fma_(e, z.im, -(mS[k2] * z.re))};
        } else {
          const cx<T> zq = get(zf[pbase - k2]);
          const cx<T> zp2 = {zq.re, -zq.im};
          T sA = mS[k2], dA = mD[k2];
          if (has_w22(t)) {
            // W22 of two columns: the loads were either column's table
            const bool w22 = f >= W::F22;
            const T sum = sA + dA, dif = sA - dA;
            sA = w22 ? sum : sA;
            dA = w22 ? dif : dA;
          }
          // (a coherence has d = 0: the same bits as the round above)
          y[k2] = {fma_(dA, zp2.im, fma_(e, z.re, sA * z.im)), fma_(-dA, zp2.re, fma_(e, z.im, -(sA * z.re)))};
        }
        if constexpr (QC) {
          // Z, Z' = the other transform of this column at m and conj at -m:
          //   packed diagonals += (c+ + i c-) Z - (c- + i c+) Z'          (Z = coherence)
          //   coherence        += (-c+ + i c-)/2 Z + (c+ + i c-)/2 Z'     (Z = packed diagonals)
          const cx<T> o = get(zo[rbase + k2]), oq = get(zo[pbase - k2]);
          const cx<T> op = {oq.re, -oq.im};
          T cp, cm;
          if constexpr (kQcEarly) {
            cp = cP[t][k2];
            cm = cM[t][k2];
          } else {
            cp = qp[k2 % MV];
            cm = qm[k2 % MV];
          }
          const T xp = hk * cp, xm = hk * cm;
          const cx<T> al = {kind ? -xp : xp, xm};
          const cx<T> be = {kind ? xp : -xm, kind ? xm : -xp};
          y[k2].re = fma_(al.re, o.re, fma_(-al.im, o.im, fma_(be.re, op.re, fma_(-be.im, op.im, y[k2].re))));
          y[k2].im = fma_(al.re, o.im, fma_(al.im, o.re, fma_(be.re, op.im, fma_(be.im, op.re, y[k2].im))));
        }
      }
      SmallDft<N2, -1, T>::run(y);
    }
    if constexpr (!QC) {
      wave_lds_sync();
      write_back(t, y);
      if (t + 1 < R2) wave_lds_sync();
    }
  }
  if constexpr (QC) {
    wave_lds_sync();
#pragma unroll
    for (int t = 0; t < R2; ++t) write_back(t, yk[t]);
  }
  wave_lds_sync();

  if constexpr (WPB > 1) issue_y();
  // second inverse pass: N1-point DFTs over stride N2, natural order out
  if constexpr (kShare1) dft16_four_lanes<-1, T>(lane, P1, N2 + 1, strided, [](int, int, cx<T> x) { return x; });
#pragma unroll
  for (int t = 0; t < (kShare1 ? 0 : R1); ++t) {
    const int item = lane + 64 * t;
    if (P1 % 64 == 0 || t + 1 < R1 || item < P1) {
      const int n2 = item % N2;
      lds_cx<T>* const z = s + item / N2 * LDP + n2;
      cx<T> x[N1];
#pragma unroll
      for (int kk = 0; kk < N1; ++kk) x[kk] = get(z[(N2 + 1) * kk]);
      SmallDft<N1, -1, T>::run(x);
#pragma unroll
      for (int n1 = 0; n1 < N1; ++n1) z[(N2 + 1) * n1] = put(x[n1]);
    }
  }
  wave_lds_sync();

  // ---- combine, write, level-0 trace partials ----------------------------
  const rsrc_t ro = make_rsrc(at(a.out, at_level), level_bytes);
  const bool want_trace = (a.partials != nullptr) && (n == 0);
  // Stores.  Left in the L2s as dirty lines, the output would be written back
  // after the last wave of the launch; written through (kStoreThrough) it
  // leaves while the launch runs, 4-9% of a mid-sized stage (us: 128 x 64 x 4 FP64,
  // four members 7.2 -> 6.6; 256 x 256 x 5 three states FP32 17.4 -> 16.0).  That
  // needs stores of whole lines: a lane's 24 or 32 bytes of FP64 nodes, written
  // through 16 at a time, cost up to 1.9x.  Where a lane has that much, the
  // wave therefore turns its columns in LDS so that each store is contiguous
  // (256 x 256 x 9 FP64 17.4 -> 16.7 one member, 205 -> 204 sixteen; 192 x 192 x 9
  // 13.45 -> 12.45 and 127 -> 120.7).
  // Past the memory-side cache (NTS, StageArgs::stream_out) they are
  // non-temporal: the next launch reads them from HBM anyway.
  constexpr bool kTurn = ES == 8 && K >= 3;
  constexpr int kPolicy = NTS ? kStoreNT : kStoreThrough;
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int q = q0 + c0l + i;
    T o[NC][K];
#pragma unroll
    for (int comp = 0; comp < NC; ++comp) {
#pragma unroll
      for (int j = 0; j < K; ++j)
        o[comp][j] = fma_(coef, loc[i][comp][j] + elem(c0l + i, comp, a0 + j), ky[i][comp][j]);
      if constexpr (!kTurn) {
        if (q < nq) buf_store_n<K, kPolicy>(o[comp], ro, qo[i + 3], comp * cbytes);
      }
    }
    if constexpr (kTurn) {
      // each lane's own nodes back to their places, other nodes out of them
      constexpr int X = K == 4 ? 2 : 1;  // nodes of a lane's second piece
      const int x0 = 2 * lig, x1 = 2 * L + X * lig;
#pragma unroll
      for (int comp = 0; comp < NC; ++comp) {
        lds_cx<T>* const z = s + W::transform(c0l + i, comp) * LDP;
        if (W::alone(comp)) {
#pragma unroll
          for (int j = 0; j < K; ++j) elem(c0l + i, comp, a0 + j) = o[comp][j];
        } else if (W::part(i, comp) == 0) {
#pragma unroll
          for (int j = 0; j < K; ++j) z[pad(a0 + j)] = lds_cx<T>{o[comp][j], o[comp + 1][j]};
        }
      }
      wave_lds_sync();
      const unsigned row = (unsigned)q * (NP * ES);
#pragma unroll
      for (int comp = 0; comp < NC; ++comp) {
        T v0[2][2], v1[2][X];
        const lds_cx<T>* const z = s + W::transform(c0l + i, comp) * LDP;
        if (!W::alone(comp) && W::part(i, comp) == 1) continue;  // (went with its real part)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const lds_cx<T> v = W::alone(comp) ? lds_cx<T>{elem(c0l + i, comp, x0 + e), T(0)} : z[pad(x0 + e)];
          v0[0][e] = v[0], v0[1][e] = v[1];
        }
#pragma unroll
        for (int e = 0; e < X; ++e) {
          const lds_cx<T> v = W::alone(comp) ? lds_cx<T>{elem(c0l + i, comp, x1 + e), T(0)} : z[pad(x1 + e)];
          v1[0][e] = v[0], v1[1][e] = v[1];
        }
#pragma unroll
        for (int c = 0; c < (W::alone(comp) ? 1 : 2); ++c)
          if (q < nq) {
            buf_store_n<2, kPolicy>(v0[c], ro, row + x0 * ES, (comp + c) * cbytes);
            buf_store_n<X, kPolicy>(v1[c], ro, row + x1 * ES, (comp + c) * cbytes);
          }
      }
    }
    if (want_trace) {
      // one partial per column, its lanes summed by a butterfly
      double tr = 0.0;
#pragma unroll
      for (int j = 0; j < K; ++j) {
#pragma unroll
        for (int u = 0; u < NS; ++u) tr = fma_(a.mu[u][u], (double)o[u][j], tr);
#pragma unroll
        for (int u = 0; u < NS; ++u)
#pragma unroll
          for (int w = u + 1; w < NS; ++w)
            tr = fma_(2.0 * a.mu[u][w], (double)o[Packing<NS>::re(u, w)][j], tr);
      }
#pragma unroll
      for (int off = L / 2; off > 0; off >>= 1) tr += __shfl_xor(tr, off, 64);
      if (lig == 0 && q < nq) a.partials[(long long)b * a.npartials + q] = tr;
    }
  }
}

// The instantiations: the shapes that wave_shape (qhfpe_internal.hpp) picks,
// each with and without members of their own depths; the largest shape of
// every np also with non-temporal stores (a constant coupling).
template <typename T, int NS, int NP, int C, int PF, int OCC, bool QC, bool NTS, int WPB>
hipError_t launch_wave_one(const StageArgs& a, int nblocks, hipStream_t s) {
  if (a.mlev)
    hipLaunchKernelGGL((stage_wave_kernel<T, NS, NP, C, PF, OCC, QC, NTS, WPB, true>), dim3(nblocks), dim3(64 * WPB), 0,
                       s, a);
  else
    hipLaunchKernelGGL((stage_wave_kernel<T, NS, NP, C, PF, OCC, QC, NTS, WPB, false>), dim3(nblocks), dim3(64 * WPB),
                       0, s, a);
  return hipGetLastError();
}

template <typename T, int NS, int NP, bool QC>
hipError_t launch_wave_np(const StageArgs& a, int nblocks, hipStream_t s) {
  // waves per SIMD: two states four in FP32 (128 VGPRs), two in FP64 or with a
  // q-dependent coupling; three states three and two; the shapes of small
  // launches, which leave SIMDs idle, as few as their loads in flight need
  constexpr bool kF32 = sizeof(T) == 4;
  constexpr int O = QC ? 2 : (NS == 2 ? (kF32 ? 4 : 2) : (kF32 ? 3 : 2));
  const WaveShape& w = a.shape;
  auto is = [&](int c, int pf, int wpb) { return w.c == c && w.pf == pf && w.wpb == wpb; };
  // (the largest shape of this np, with the stores of StageArgs::stream_out)
#define QHFPE_LARGEST(C, PF, WPB)                                                                      \
  if (is(C, PF, WPB)) {                                                                                \
    if constexpr (!QC) {                                                                               \
      if (a.stream_out) return launch_wave_one<T, NS, NP, C, PF, O, QC, true, WPB>(a, nblocks, s);     \
    }                                                                                                  \
    return launch_wave_one<T, NS, NP, C, PF, O, QC, false, WPB>(a, nblocks, s);                        \
  }
#define QHFPE_SHAPE(C, PF, OCC, WPB) \
  if (is(C, PF, WPB)) return launch_wave_one<T, NS, NP, C, PF, OCC, QC, false, WPB>(a, nblocks, s);
  if constexpr (NS == 2) {
    QHFPE_SHAPE(1, 2, 2, 1)
    if constexpr (kF32 && !QC) QHFPE_SHAPE(1, 4, 1, 1)
    if constexpr (NP == 256 && kF32 && !QC) {
      QHFPE_SHAPE(2, 1, O, 2)
      QHFPE_LARGEST(2, 1, 4)
    } else if constexpr (NP == 256) {
      QHFPE_SHAPE(2, kStaggered, O, 2)
      QHFPE_LARGEST(2, kStaggered, 4)
    } else if constexpr (NP == 192) {
      QHFPE_LARGEST(2, kStaggered, 4)
    } else if constexpr (NP == 128 || NP == 64) {
      QHFPE_SHAPE(2, kStaggered, O, 2)
      QHFPE_LARGEST(4, kStaggered, 4)
    } else {
      QHFPE_LARGEST(2, kStaggered, 2)
    }
  } else {
    if constexpr (kF32 || NP == 128 || NP == 64) QHFPE_SHAPE(1, 3, 2, 1)
    if constexpr (NP == 128 || NP == 64) {
      QHFPE_SHAPE(1, kStaggered, O, 2)
      QHFPE_LARGEST(2, kStaggered, 2)
    } else {
      QHFPE_LARGEST(1, kStaggered, 2)
    }
  }
#undef QHFPE_SHAPE
#undef QHFPE_LARGEST
  return hipErrorInvalidValue;
}

template <typename T, int NS>
hipError_t launch_stage_wave(int np, const StageArgs& a, int nblocks, hipStream_t s) {
  switch (np) {
#define QHFPE_CASE(NP_)                                                       \
  case NP_:                                                                   \
    if constexpr (NS == 2) {                                                  \
      if (a.qcoup) return launch_wave_np<T, NS, NP_, true>(a, nblocks, s);    \
    }                                                                         \
    return launch_wave_np<T, NS, NP_, false>(a, nblocks, s);
    QHFPE_CASE(32)
    QHFPE_CASE(48)
    QHFPE_CASE(64)
    QHFPE_CASE(96)
    QHFPE_CASE(128)
    QHFPE_CASE(192)
    QHFPE_CASE(256)
#undef QHFPE_CASE
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace qhfpe
