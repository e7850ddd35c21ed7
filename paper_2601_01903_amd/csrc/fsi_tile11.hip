// Register-phase tile kernel of the fused FSI algorithm (gfx950), tiles of
// 2^11 values, l <= 4.
//
// A workgroup of 256 threads owns a work item: a run of tiles of one
// instance (raw v, high index U_H) and one group of its outputs. Per tile it
// computes
//   - the in-tile Moebius butterfly (Sec. 4.2) over the 11 low bits: bits
//     8-10 in registers straight from the coalesced loads, bits 4-7 and 0-3
//     through two LDS transposes;
//   - the left-to-right counter sweep (Sec. 4.3 - 4.4) in three phases of 4,
//     4 and 3 sites. Within a phase a thread owns one output prefix with all
//     its counters and the phase's 2^P inputs in registers and walks the
//     phase's output bits depth first: each output state adds its tau = 0
//     and tau = 1 predecessors (the sparse MPO cores). Between phases the
//     (sigma, t) states go through LDS, truncated to |sigma| <= l (the
//     compressed output prefix). Phase B splits its first output site
//     between the two halves of the workgroup (sigma = 0 and sigma = 1
//     subtrees); phase C splits it for its heavy prefixes only. Threads are
//     ordered so that each wave's prefixes share bounds on their popcount,
//     and each wave runs code compiled for those bounds;
//   - the final weight core with the Moebius cores of the high sites
//     precontracted into it (Sec. 4.5 applied to the high sites), in FP64:
//     Y[S_L, s_H, j] = sum_t lambda_u(s_L + s_H, t, s_H + u - j) Z[S_L, t],
//     u = |U_H|; a wave first loads the Z rows of all its tasks, then
//     computes them; rows of one |S_L| take wave-uniform weights through
//     scalar loads, the (row, slot) pairs of |S_L| <= 1 per-lane weights
//     staged in LDS;
//   - the cross-tile sum E_S += Y[S_L, |S_H|, |S_H & U_H|] in FP64 registers
//     for the outputs of the item's group.
// At the end of the item the FP64 partial sums go to a workspace; the
// reduction kernel adds the items of an instance in a fixed order. An
// instance of one item writes its scores itself, so a plan of such instances is
// one launch.
//
// Every LDS layout is a compile-time function of l (fsi_tile11.h), so the
// hot loops address LDS with one per-thread base register and immediate
// offsets. LDS regions:
//   region 1: raw-tile transposes and, after them, the partial results Y;
//             phase-B states S2 overlay both (no barrier between a tile's
//             gather and the next tile's loads)
//   region 2: phase-A states S1 -> final states Z
//   region 3: the final-core weights of the current |U_H| (per-lane reads
//             of the |S_L| <= 1 pairs)
//   a zero row read in place of counter rows past a unit's range
// The forms of l = 3 that share a CU overlay regions 1 and 2 (struct Lds).
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "fsi_kernels.h"
#include "fsi_sweep_dev.h"
#include "fsi_tile11.h"

namespace fsi {
namespace t11 {

// --------------------------------------------------------------- LDS plan
constexpr int align256(int x) { return (x + 255) & ~255; }
constexpr int imax2(int a, int b) { return a > b ? a : b; }
// Gather positions a kernel of order L is compiled for: few of them (the
// accumulators of the larger instances cost registers, and with them
// workgroups per CU) or the most its outputs need.
constexpr int np_few(int L) { return L == 3 ? 4 : L == 4 ? 7 : np_order(L); }
constexpr int np_compiled(int L, int np) { return np <= np_few(L) ? np_few(L) : np_order(L); }

// Workgroups per CU (4 waves each, one per SIMD) the registers are held to.
// FP32 sweep: 3 at l <= 2 and, with few accumulators, at l = 3 (168 VGPRs),
// else 2 (256); FP64: 2 at l <= 2 and l = 3 with few accumulators, else 1
// (LDS at l = 4, registers at l = 3).
template <typename SwT> constexpr int wgs_of(int L, int NP) {
  const bool light = L <= 2 || (L == 3 && NP <= np_few(3));
  return sizeof(SwT) == 4 ? (light ? 3 : 2) : (light ? 2 : 1);
}
// Whether the sweep's phases share one region (each phase's inputs in
// registers, a barrier, then its stores over them): where the separate
// regions do not leave room for wgs_of workgroups.
template <typename SwT> constexpr bool shared_of(int L, int NP) {
  return L == 3 && NP <= np_few(3);
}

template <int L, typename SwT, typename MobT, bool SHARED>
struct Lds {
  static constexpr int rend = align256((int)(r_elems * sizeof(MobT)));
  static constexpr int s1b = rows1(L) * row1_stride<SwT>() * (int)sizeof(SwT);
  static constexpr int s2b = s2_elems(L) * (int)sizeof(SwT);
  static constexpr int zb = align256((nzrows(L) + 1) * ZROW * (int)sizeof(SwT));
  static constexpr int yb = ysize(L) * 8;
  // separate: region 1 holds the raw-tile transposes at 0 and the partial
  // results Y after them (disjoint, so the next tile's loads and first
  // transpose may start while slower waves still gather this tile's Y), and
  // phase B's states S2 over both; region 2 S1, then Z.
  // shared: the transposes at 0, S1 after them, S2 over both, Z over S2, Y
  // past Z and the transposes.
  static constexpr int yoff = SHARED ? imax2(rend, zb) : rend;
  static constexpr int reg1 = align256(SHARED ? imax2(rend + s1b, imax2(s2b, yoff + yb))
                                              : imax2(s2b, yoff + yb));
  static constexpr int s1off = SHARED ? rend : reg1;
  static constexpr int zoff = SHARED ? 0 : reg1;
  static constexpr int reg2 = SHARED ? 0 : align256(imax2(s1b, zb));
  static constexpr int reg3 = align256(lamblock(L) * 8);   // weights of the current |U_H|
  static constexpr int lamoff_ = reg1 + reg2;
  static constexpr int end = reg1 + reg2 + reg3;
};
// Past the regions: zeros, read in place of the counter rows past a prefix's
// range by the waves that run the general sweep code (their row loads then
// need no branch and issue back to back), and the words that lanes past a
// weight task's rows write.
constexpr int kLdsZeros = 128, kLdsTail = kLdsZeros + 128;
// A kernel of one order places them at that order's end; the kernel that runs
// items of every order at one offset past the regions of all of them.
template <typename SwT, typename MobT>
struct LdsAll {
  static constexpr int end =
      imax2(imax2(Lds<1, SwT, MobT, false>::end, Lds<2, SwT, MobT, false>::end),
            imax2(Lds<3, SwT, MobT, false>::end, Lds<4, SwT, MobT, false>::end));
};

// ------------------------------------------------------------ weight core
// Row task: 64 lanes, each owning one Z row of |S_L| = S (S >= 2) and
// producing the slots [K0, K1) of it; the weights are the same for every
// lane. Pair task: the (row, slot) pairs of |S_L| <= 1, 64 per task, with
// per-lane weights.
// Compile-time schedule of the weight-core tasks of one tile over the four
// waves (longest task first to the least loaded wave). Row tasks of rows
// with many slots are split into two slot ranges.
struct LamTask { int kind, S, chunk, k0, k1, cost, wave; };
struct LamPlan { LamTask t[40]; int n; };
constexpr LamPlan make_lam_plan(int L) {
  LamPlan p{};
  p.n = 0;
  for (int S = L; S >= 2; --S) {
    const int RC = ZROW - S, NS = nslots(L, S);
    for (int c = 0; c < row_tasks(S); ++c) {
      const int parts = NS * RC > 40 ? 2 : 1;
      for (int q = 0; q < parts; ++q) {
        const int k0 = NS * q / parts, k1 = NS * (q + 1) / parts;
        p.t[p.n++] = LamTask{0, S, c, k0, k1, (k1 - k0) * RC + RC + 8, -1};
      }
    }
  }
  for (int c = 0; c < (npairs(L) + 63) / 64; ++c) p.t[p.n++] = LamTask{1, 0, c, 0, 0, 2 * ZROW + 8, -1};
  int load[NT / 64] = {0, 0, 0, 0};
  for (int done = 0; done < p.n; ++done) {
    int best = -1;
    for (int i = 0; i < p.n; ++i)
      if (p.t[i].wave < 0 && (best < 0 || p.t[i].cost > p.t[best].cost)) best = i;
    int w = 0;
    for (int q = 1; q < NT / 64; ++q)
      if (load[q] < load[w]) w = q;
    p.t[best].wave = w;
    load[w] += p.t[best].cost;
  }
  return p;
}
template <int L> struct LP { static constexpr LamPlan plan = make_lam_plan(L); };


// Tasks of one wave in plan order, with the offset of each task's Z row in
// the wave's register buffer.
struct WaveList { int idx[40]; int n; };
constexpr WaveList make_wave_list(int L, int W) {
  WaveList w{};
  w.n = 0;
  const LamPlan p = make_lam_plan(L);
  for (int i = 0; i < p.n; ++i)
    if (p.t[i].wave == W) w.idx[w.n++] = i;
  return w;
}
template <int L, int W> struct WL { static constexpr WaveList w = make_wave_list(L, W); };

// Pass 1: every Z row (and the per-lane weights of pair tasks) of the
// wave's tasks is loaded before any arithmetic, so the LDS latency is paid
// once per tile.
template <int L, int W, int J, typename SwT>
__device__ __forceinline__ void lam_load(int lane, const SwT* Z, const double* lam,
                                         SwT (&zb)[ZROW * (WL<L, W>::w.n > 0 ? WL<L, W>::w.n : 1)],
                                         double (&pw)[ZROW * 2]) {
  if constexpr (J < WL<L, W>::w.n) {
    constexpr LamTask T = LP<L>::plan.t[WL<L, W>::w.idx[J]];
    using V = typename Vec4<SwT>::type;
    constexpr int VN = Vec4<SwT>::n;
    const SwT* zr;
    if constexpr (T.kind == 0) {
      constexpr int NR = cbinom(B, T.S);
      constexpr bool full = (T.chunk + 1) * 64 <= NR;
      const int row = T.chunk * 64 + lane;
      zr = Z + (zbase(T.S) + (full || row < NR ? row : 0)) * ZROW;
    } else {
      constexpr int N0 = nslots(L, 0), N1 = nslots(L, 1);
      const int p0 = T.chunk * 64 + lane;
      const int p = p0 < K<L>::NPAIR ? p0 : 0;
      const bool z0 = p < N0;
      const int row = (p - N0) / N1, slot = (p - N0) - row * N1;
      zr = Z + (z0 ? 0 : 1 + row) * ZROW;
      const int lofs = z0 ? K<L>::LAM0 + p * ZROW : K<L>::LAM1 + slot * ZROW;
      const double2* lw = reinterpret_cast<const double2*>(lam + lofs);
      constexpr int PB = (T.chunk & 1) * ZROW;   // at most two pair tasks per wave
#pragma unroll
      for (int q = 0; q < ZROW / 2; ++q) {
        const double2 w = lw[q];
        pw[PB + 2 * q] = w.x;
        pw[PB + 2 * q + 1] = w.y;
      }
    }
    const V* zv = reinterpret_cast<const V*>(zr);
    // a row task reads only its counters (12 - |S_L| entries)
    constexpr int NV = T.kind == 0 ? (ZROW - T.S + VN - 1) / VN : ZROW / VN;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const V v = zv[q];
      if constexpr (VN == 4) {
        zb[J * ZROW + 4 * q] = v.x; zb[J * ZROW + 4 * q + 1] = v.y;
        zb[J * ZROW + 4 * q + 2] = v.z; zb[J * ZROW + 4 * q + 3] = v.w;
      } else {
        zb[J * ZROW + 2 * q] = v.x; zb[J * ZROW + 2 * q + 1] = v.y;
      }
    }
    lam_load<L, W, J + 1, SwT>(lane, Z, lam, zb, pw);
  }
}

// Pass 2: the slots of every task. Row tasks take their weights from the
// constant address space (wave-uniform: scalar loads); lanes past the last
// row write to a dump word.
template <int L, int W, int J, typename SwT>
__device__ __forceinline__ void lam_comp(int lane, double* Y, cdptr lamg, double* dump,
                                         const SwT (&zb)[ZROW * (WL<L, W>::w.n > 0 ? WL<L, W>::w.n : 1)],
                                         const double (&pw)[ZROW * 2]) {
  if constexpr (J < WL<L, W>::w.n) {
    constexpr LamTask T = LP<L>::plan.t[WL<L, W>::w.idx[J]];
    if constexpr (T.kind == 0) {
      constexpr int S = T.S, K0 = T.k0, K1 = T.k1;
      constexpr int NR = cbinom(B, S);
      constexpr int RC = ZROW - S;
      constexpr int LO = lamoff(L, S), YB = ybase(L, S);
      constexpr bool full = (T.chunk + 1) * 64 <= NR;
      const int row = T.chunk * 64 + lane;
      double z[RC];
#pragma unroll
      for (int r = 0; r < RC; ++r) z[r] = (double)zb[J * ZROW + r];
      double a[K1 - K0];
#pragma unroll
      for (int k = K0; k < K1; ++k) a[k - K0] = 0.0;
#pragma unroll
      for (int r = 0; r < RC; ++r)
#pragma unroll
        for (int k = K0; k < K1; ++k) a[k - K0] = fma(lamg[LO + k * ZROW + r], z[r], a[k - K0]);
      const bool ok = full || row < NR;
#pragma unroll
      for (int k = K0; k < K1; ++k) *(ok ? Y + YB + k * nrp(S) + row : dump) = a[k - K0];
    } else {
      constexpr int N0 = nslots(L, 0), N1 = nslots(L, 1);
      constexpr int PB = (T.chunk & 1) * ZROW;
      const int p0 = T.chunk * 64 + lane;
      const bool ok = p0 < K<L>::NPAIR;
      const int p = ok ? p0 : 0;
      const bool z0 = p < N0;
      const int row = (p - N0) / N1, slot = (p - N0) - row * N1;
      const int yidx = z0 ? K<L>::YB0 + p * nrp(0) : K<L>::YB1 + slot * nrp(1) + row;
      double a = 0.0;
#pragma unroll
      for (int r = 0; r < ZROW; ++r) {
        // entry 11 of an |S_L| = 1 row lies past its counters (weight 0)
        const double zz = (r < ZROW - 1 || z0) ? (double)zb[J * ZROW + r] : 0.0;
        a = fma(pw[PB + r], zz, a);
      }
      *(ok ? Y + yidx : dump) = a;
    }
    lam_comp<L, W, J + 1, SwT>(lane, Y, lamg, dump, zb, pw);
  }
}

template <int L, int W, typename SwT>
__device__ __forceinline__ void lam_wave(int lane, const SwT* Z, double* Y, const double* lam,
                                         cdptr lamg, double* dump) {
  SwT zb[ZROW * (WL<L, W>::w.n > 0 ? WL<L, W>::w.n : 1)];
  double pw[ZROW * 2];
  lam_load<L, W, 0, SwT>(lane, Z, lam, zb, pw);
  lam_comp<L, W, 0, SwT>(lane, Y, lamg, dump, zb, pw);
}

// ---------------------------------------------------------- wave priority
// Two workgroups share each SIMD (one wave of each). Within a step separated
// by barriers the waves' shares of the work differ; the wave with the
// longest share is issued first (s_setprio), so the other workgroup's waves
// fill the idle cycles instead of delaying that step's slowest wave.
template <int P> __device__ __forceinline__ void wave_prio() { __builtin_amdgcn_s_setprio(P); }
// phase B: (half 0, low |sigma_A|) > (half 0, high) > (half 1, low) > (half 1, high)
constexpr int kPrioB[NT / 64] = {3, 2, 1, 0};
// phase C: heavy sigma = 0 subtrees > low-|sigma_AB| whole trees > heavy
// sigma = 1 subtrees > the rest
constexpr int prio_c(int w) {
  return w == kCWaveH0 ? 3 : w == kCWaveR0 ? 2 : w == kCWaveH1 ? 1 : 0;
}
// the two-wave Moebius steps run ahead of the idle waves' next step; the
// weight core and the gather (every wave an equal share) stay at 0, behind
// the sweep steps of the other workgroup
constexpr int kPrioTwoWave = 1;

// ------------------------------------------------------------------ item
// TAIL: LDS offset of the zeros. NPC: gather positions.
template <int L, typename SwT, typename MobT, bool IN64, bool MOBIN, int NPC, bool SHARED, int TAIL>
__device__ __forceinline__ void run_item(const FastClassDev* __restrict__ C, const InstDev& I,
                                         const FastItem& W, const float* __restrict__ vals32,
                                         const double* __restrict__ vals64,
                                         const int32_t* __restrict__ torder,
                                         double* __restrict__ partial,
                                         void* __restrict__ out, unsigned char* smem) {
  static_assert(kFastRuns == kRuns, "gather positions");
  constexpr int NP = NPC;             // gather positions
  constexpr int KMAX = 2 * NP;        // output slots
  constexpr int LB = K<L>::LB;
  using LD = Lds<L, SwT, MobT, SHARED>;
  MobT* R = reinterpret_cast<MobT*>(smem);
  SwT* S2 = reinterpret_cast<SwT*>(smem);
  double* Y = reinterpret_cast<double*>(smem + LD::yoff);
  SwT* S1 = reinterpret_cast<SwT*>(smem + LD::s1off);
  SwT* Z = reinterpret_cast<SwT*>(smem + LD::zoff);
  double* lamL = reinterpret_cast<double*>(smem + LD::lamoff_);
  const SwT* zrow = reinterpret_cast<const SwT*>(smem + TAIL);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- per-item thread constants ----
  // phase B: thread (half, rankA, c); half = tid / 128 is wave-uniform
  // (waves 0, 2: sigma_A ranks 0-7; waves 1, 3: ranks 8-15)
  const int p2r = (((tid & 127) >> 6) << 3) | (tid & 7), p2c = (tid >> 3) & 7;
  const int sA_mask = (int)((kOrderANibbles >> (4 * p2r)) & 15u);
  const int sA = __popc(sA_mask);
  const int wb = ((p2c >> 2) * K<L>::S2U + p2r) * 4 + (p2c & 3);
  // phase C: thread = unit
  const int u3r = C->uperm[tid];
  const bool c_on = u3r >= 0;   // this thread has a phase-C unit
  const int u3 = c_on ? u3r : 0;
  int sAB = __popc(C->unit_mask[u3]);
  int zr[NC];
#pragma unroll
  for (int sc = 0; sc < NC; ++sc) zr[sc] = C->zrow[u3 * NC + sc];
  if (SHARED && !c_on) {   // runs unit 0 into the dump row
    sAB = KAB;
#pragma unroll
    for (int sc = 0; sc < NC; ++sc) zr[sc] = nzrows(L);
  }
  // cross-tile sum (the output metadata is re-read per tile from L1/L2 so it
  // holds no registers during the sweep phases)
  double acc[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) acc[k] = 0.0;
  const uint4* meta_g = reinterpret_cast<const uint4*>(C->meta + (size_t)tid * kFastMetaStride);
  // j-stride of Y per (position, wave)
  const cdptr_u gs8 = (cdptr_u)(C->gs8 + wave);
  const int nkk = C->nkk;
  // input already Moebius-transformed (a separate instantiation): the
  // butterflies are skipped
  constexpr bool mob = !MOBIN;
  const int mshift = C->mshift;
  const uint32_t omask = (1u << mshift) - 1u;
  int u_prev = -1;

  const int64_t vbase = I.voff;
  using RawT = typename std::conditional<IN64, double, float>::type;
  RawT xraw[NC];   // next tile's raw values (converted when its butterfly starts)
  // an instance with d < 11 (lowmask = 2^d - 1) runs as d = 11: the value
  // of U is v(U & lowmask), and its Moebius coefficients past bit d - 1
  // are zero (Moebius input)
  const int lowmask = I.lowmask;
  auto load_tile = [&](int UH) {
    const int64_t base = vbase + ((int64_t)UH << B);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int idx = tid + (c << 8);
      const int64_t at = base + (idx & lowmask);
      if constexpr (MOBIN) {
        if constexpr (IN64) xraw[c] = idx <= lowmask ? vals64[at] : 0.0;
        else xraw[c] = idx <= lowmask ? vals32[at] : 0.f;
      } else {
        if constexpr (IN64) xraw[c] = vals64[at];
        else xraw[c] = vals32[at];
      }
    }
  };
  int UH = torder[I.tofs + W.tb];
  load_tile(UH);

  for (int k = W.tb; k < W.te; ++k) {
    const int UHn = k + 1 < W.te ? torder[I.tofs + k + 1] : 0;
    const int u = __builtin_amdgcn_readfirstlane(__popc(UH));
    if (u != u_prev) {
      // tiles run in order of |U_H|: the weights change at most h + 1 times
      const double* src = C->lam + (int64_t)u * LB;
      for (int i = tid; i < LB; i += NT) lamL[i] = src[i];
      u_prev = u;
    }

    // ---- Moebius over bits 8-10 in registers, then transpose (ahead of
    // the other workgroup's weight core and gather) ----
    wave_prio<1>();
    MobT xr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if constexpr (IN64) xr[c] = mob_from_d<MobT>(xraw[c]);
      else xr[c] = mob_from<MobT>(xraw[c]);
    }
    if (mob) {
#pragma unroll
      for (int bit = 0; bit < PC; ++bit)
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (c & (1 << bit)) xr[c] = sub(xr[c], xr[c ^ (1 << bit)]);
    }
    {
      MobT* rp = R + (tid & 15) + RB * (tid >> 4);
#pragma unroll
      for (int c = 0; c < NC; ++c) rp[RC_ * c] = xr[c];
    }
    wave_prio<0>();
    __syncthreads();
    // ---- Moebius over bits 4-7: thread (a, c) holds the 16 b values ----
    if (tid < NA * NC) {
      wave_prio<kPrioTwoWave>();
      MobT* rp = R + (tid & 15) + RC_ * (tid >> 4);
      MobT y[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) y[b] = rp[RB * b];
      if (mob) {
#pragma unroll
        for (int bit = 0; bit < PB; ++bit)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            if (b & (1 << bit)) y[b] = sub(y[b], y[b ^ (1 << bit)]);
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) rp[RB * b] = y[b];
      wave_prio<0>();
    }
    __syncthreads();
    // ---- Moebius over bits 0-3 + phase A: thread (b, c) of waves 2-3 holds
    // the 16 a values (waves 0-1 ran the B bits: the two-wave steps are
    // spread over all four SIMDs) ----
    if (tid >= NT - NB * NC) {
      wave_prio<kPrioTwoWave>();
      const int ta = tid - (NT - NB * NC);
      const MobT* rp = R + RB * (ta & 15) + RC_ * (ta >> 4);
      MobT y[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) y[a] = rp[a];
      if (mob) {
#pragma unroll
        for (int bit = 0; bit < PA; ++bit)
#pragma unroll
          for (int a = 0; a < NA; ++a)
            if (a & (1 << bit)) y[a] = sub(y[a], y[a ^ (1 << bit)]);
      }
      SwT X1[1][NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) X1[0][a] = to_sw<SwT>(y[a]);
      EmitS1<SwT, L> e1{S1 + ta};
      rsweep<PA, 0, 1, 0>(X1, e1);
      wave_prio<0>();
    }
    __syncthreads();
    // ---- phase B: thread (half, sigma_A, c), counters relative to |sigma_A|;
    // the first output site (b bit 3) is split between the two halves of the
    // workgroup: half 0 walks the sigma = 0 subtree, half 1 the sigma = 1
    // subtree (which needs only the tau = 1 inputs); in each half the second
    // wave holds the sigma_A with |sigma_A| >= 2 ----
    switch (wave) {
      case 0:
        wave_prio<kPrioB[0]>();
        phase_b<L, 0, kSALoMax, 0, SwT, SHARED>(S1, S2 + wb, sA, p2r, p2c);
        break;
      case 1:
        wave_prio<kPrioB[1]>();
        phase_b<L, kSAHi, kSAHiMax, 0, SwT, SHARED>(S1, S2 + wb, sA, p2r, p2c);
        break;
      case 2:
        wave_prio<kPrioB[2]>();
        phase_b<L, 0, kSALoMax, 1, SwT, SHARED>(S1, S2 + wb, sA, p2r, p2c);
        break;
      default:
        wave_prio<kPrioB[3]>();
        phase_b<L, kSAHi, kSAHiMax, 1, SwT, SHARED>(S1, S2 + wb, sA, p2r, p2c);
        break;
    }
    wave_prio<0>();
    __syncthreads();
    // ---- phase C: thread per unit sigma_AB (units in order of |sigma_AB|,
    // the heavy ones split between two waves), counters relative to
    // |sigma_AB| ----
    // (shared region: every thread runs it, for its barrier)
    if (c_on || SHARED) {
      using O = UO<L>;
      switch (wave) {
        case 0:
          wave_prio<prio_c(0)>();
          phase_c<L, O::o.kmin[0], O::o.kmax[0], O::o.part[0], SwT, SHARED>(S2, Z, zr, sAB, u3, zrow);
          break;
        case 1:
          wave_prio<prio_c(1)>();
          phase_c<L, O::o.kmin[1], O::o.kmax[1], O::o.part[1], SwT, SHARED>(S2, Z, zr, sAB, u3, zrow);
          break;
        case 2:
          wave_prio<prio_c(2)>();
          phase_c<L, O::o.kmin[2], O::o.kmax[2], O::o.part[2], SwT, SHARED>(S2, Z, zr, sAB, u3, zrow);
          break;
        default:
          wave_prio<prio_c(3)>();
          phase_c<L, O::o.kmin[3], O::o.kmax[3], O::o.part[3], SwT, SHARED>(S2, Z, zr, sAB, u3, zrow);
          break;
      }
      wave_prio<0>();
    }
    // prefetch the next tile and this tile's output metadata while the
    // weight core runs
    if (k + 1 < W.te) load_tile(UHn);
    uint32_t meta[(NP + 3) & ~3];
#pragma unroll
    for (int q = 0; q < (NP + 3) / 4; ++q) {
      const uint4 v = meta_g[q];
      meta[4 * q] = v.x; meta[4 * q + 1] = v.y; meta[4 * q + 2] = v.z; meta[4 * q + 3] = v.w;
    }
    __syncthreads();
    // ---- final weight core -> Y ----
    {
      const cdptr lamg = (cdptr)(C->lam + (int64_t)u_prev * LB);
      double* dump = reinterpret_cast<double*>(smem + TAIL + kLdsZeros);
      switch (wave) {
        case 0: lam_wave<L, 0, SwT>(lane, Z, Y, lamL, lamg, dump); break;
        case 1: lam_wave<L, 1, SwT>(lane, Z, Y, lamL, lamg, dump); break;
        case 2: lam_wave<L, 2, SwT>(lane, Z, Y, lamL, lamg, dump); break;
        default: lam_wave<L, 3, SwT>(lane, Z, Y, lamL, lamg, dump); break;
      }
    }
    __syncthreads();
    // ---- cross-tile sum: E_S += Y[S_L, s_H, |S_H & U_H|] ----
    // position p holds a run of two outputs (ranks 2r, 2r + 1 of one |S_L|,
    // one S_H): one popcount and one 16-byte read; the j-stride is uniform
    // in the wave
    {
      const uint32_t UHs = (uint32_t)UH << mshift;
      const unsigned char* Yb = reinterpret_cast<const unsigned char*>(Y);
      constexpr int GB = 5;   // runs per batch of reads
#pragma unroll
      for (int p0 = 0; p0 < NP; p0 += GB) {
        double2 v[GB];
#pragma unroll
        for (int q = 0; q < GB; ++q) {
          if (p0 + q < NP) {
            const uint32_t m = meta[p0 + q];
            const uint32_t off = (m & omask) + (uint32_t)__popc(m & UHs) * gs8[(p0 + q) * 4];
            v[q] = *reinterpret_cast<const double2*>(Yb + off);
          }
        }
#pragma unroll
        for (int q = 0; q < GB; ++q)
          if (p0 + q < NP) {
            acc[2 * (p0 + q)] += v[q].x;
            acc[2 * (p0 + q) + 1] += v[q].y;
          }
      }
    }
    UH = UHn;
    // no barrier: the next tile's first writes (the transpose region, and
    // the weights once every wave has passed the barrier before this
    // gather) do not touch Y
  }
  // ---- the item's sums ----
  using OutT = RawT;   // the storage type
  if (I.fold) {
    // the instance's only item: its sums are the scores (a single apply at
    // d <= 11 is one launch: 13 -> 11 us back to back). Adding a few items
    // here too, by the last one to end, cost more than the reduction's launch:
    // its device-wide fences took d = 14 from 15 to 20 us and 512 uneven
    // instances from 390 to 485 us.
    OutT* o = static_cast<OutT*>(out) + I.ooff;
#pragma unroll
    for (int kk = 0; kk < KMAX; ++kk)
      if (kk < nkk) {
        const int q = I.sinv[kk * NT + tid];
        if (q >= 0) o[q] = (OutT)acc[kk];
      }
    return;
  }
  double* P = partial + W.pofs + tid;
#pragma unroll
  for (int kk = 0; kk < KMAX; ++kk)
    if (kk < nkk) P[kk * NT] = acc[kk];
}

// Work queue of a launch: workgroup b runs item b first, then takes the
// next unclaimed item (from gridDim.x on) each time it is done, so items of
// unequal cost (instances of different d and l in one batch) spread over the
// machine as they finish (items are sorted by decreasing cost). queue[0]
// counts the items taken after the first round, queue[1] the workgroups
// that found the queue empty; the last of those clears both for the next
// launch on the stream. A launch with no more items than workgroups does
// not touch the queue. No fence: a workgroup's add to queue[0] has returned
// before it adds to queue[1], so the last one finds every add done, and the
// end of the launch makes the zeros visible (a fence per workgroup writes the
// XCD's L2 back: 4 to 10 us a launch, 512 ragged instances 371 -> 362 us).
__device__ __forceinline__ int next_item(uint32_t* queue, int n_items) {
  if (n_items <= (int)gridDim.x) return n_items;
  __shared__ int s_item;
  if (threadIdx.x == 0) s_item = (int)(gridDim.x + atomicAdd(queue, 1u));
  __syncthreads();
  return s_item;
}
__device__ __forceinline__ void queue_done(uint32_t* queue, int n_items) {
  if (n_items > (int)gridDim.x && threadIdx.x == 0) {
    if (atomicAdd(queue + 1, 1u) == gridDim.x - 1) {
      atomicExch(queue, 0u);
      atomicExch(queue + 1, 0u);
    }
  }
}

// One kernel per order l (the items of a launch all have that order).
template <int L, typename SwT, typename MobT, bool IN64, bool MOBIN, int NP>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(wgs_of<SwT>(L, NP))))
tile11_kernel(const FastClassDev* __restrict__ classes, const InstDev* __restrict__ insts,
              const FastItem* __restrict__ items, int n_items,
              const float* __restrict__ vals32, const double* __restrict__ vals64,
              const int32_t* __restrict__ torder, double* __restrict__ partial,
              void* __restrict__ out, uint32_t* __restrict__ queue) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr bool SHARED = shared_of<SwT>(L, NP);
  constexpr int TAIL = Lds<L, SwT, MobT, SHARED>::end;
  if (threadIdx.x < kLdsZeros / 4) reinterpret_cast<uint32_t*>(smem + TAIL)[threadIdx.x] = 0u;
  __syncthreads();
  for (int item = blockIdx.x; item < n_items; item = next_item(queue, n_items)) {
    const FastItem W = items[item];
    const InstDev I = insts[W.inst];
    run_item<L, SwT, MobT, IN64, MOBIN, NP, SHARED, TAIL>(classes + I.fcls, I, W, vals32, vals64,
                                                          torder, partial, out, smem);
    __syncthreads();
  }
  queue_done(queue, n_items);
}

// Items of every order in one launch (a batch of instances with different
// l): each item runs the code compiled for its instance's order; the
// regions of all orders share one allocation (LdsAll).
template <typename SwT, typename MobT, bool IN64, bool MOBIN>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(SwT) == 4 ? 2 : 1)))
tile11_mixed_kernel(const FastClassDev* __restrict__ classes, const InstDev* __restrict__ insts,
                    const FastItem* __restrict__ items, int n_items,
                    const float* __restrict__ vals32, const double* __restrict__ vals64,
                    const int32_t* __restrict__ torder, double* __restrict__ partial,
                    void* __restrict__ out, uint32_t* __restrict__ queue) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int TAIL = LdsAll<SwT, MobT>::end;
  if (threadIdx.x < kLdsZeros / 4) reinterpret_cast<uint32_t*>(smem + TAIL)[threadIdx.x] = 0u;
  __syncthreads();
  for (int item = blockIdx.x; item < n_items; item = next_item(queue, n_items)) {
    const FastItem W = items[item];
    const InstDev I = insts[W.inst];
    const FastClassDev* C = classes + I.fcls;
    const int l = __builtin_amdgcn_readfirstlane(C->l);
    switch (l) {
      case 1: run_item<1, SwT, MobT, IN64, MOBIN, np_order(1), false, TAIL>(C, I, W, vals32, vals64, torder, partial, out, smem); break;
      case 2: run_item<2, SwT, MobT, IN64, MOBIN, np_order(2), false, TAIL>(C, I, W, vals32, vals64, torder, partial, out, smem); break;
      case 3: run_item<3, SwT, MobT, IN64, MOBIN, np_order(3), false, TAIL>(C, I, W, vals32, vals64, torder, partial, out, smem); break;
      default: run_item<4, SwT, MobT, IN64, MOBIN, np_order(4), false, TAIL>(C, I, W, vals32, vals64, torder, partial, out, smem); break;
    }
    __syncthreads();
  }
  queue_done(queue, n_items);
}

}  // namespace t11

using namespace t11;

// ------------------------------------------------------------------ launcher
// Kernel, LDS bytes and workgroups per CU of one form.
struct FastForm {
  const void* fn;
  int lds, wgs;
};
constexpr int lds_wgs(int lds, int wgs) {
  const int by_lds = 160 * 1024 / lds;
  return by_lds < 1 ? 1 : by_lds < wgs ? by_lds : wgs;
}
template <int L, typename SwT, typename MobT, bool IN64, bool MOBIN, int NP>
static FastForm form_np() {
  constexpr int lds = Lds<L, SwT, MobT, shared_of<SwT>(L, NP)>::end + kLdsTail;
  static_assert(lds <= 160 * 1024, "register-phase kernel does not fit in LDS");
  return FastForm{reinterpret_cast<const void*>(tile11_kernel<L, SwT, MobT, IN64, MOBIN, NP>), lds,
                  lds_wgs(lds, wgs_of<SwT>(L, NP))};
}
template <int L, typename SwT, typename MobT, bool IN64, bool MOBIN>
static FastForm form_l(int np) {
  if constexpr (np_few(L) != np_order(L))
    if (np <= np_few(L)) return form_np<L, SwT, MobT, IN64, MOBIN, np_few(L)>();
  return form_np<L, SwT, MobT, IN64, MOBIN, np_order(L)>();
}
template <typename SwT, typename MobT, bool IN64, bool MOBIN>
static FastForm form_t(int l, int np) {
  switch (l) {
    case 1: return form_l<1, SwT, MobT, IN64, MOBIN>(np);
    case 2: return form_l<2, SwT, MobT, IN64, MOBIN>(np);
    case 3: return form_l<3, SwT, MobT, IN64, MOBIN>(np);
    case 4: return form_l<4, SwT, MobT, IN64, MOBIN>(np);
  }
  constexpr int lds = LdsAll<SwT, MobT>::end + kLdsTail;   // l = 0: every order
  return FastForm{reinterpret_cast<const void*>(tile11_mixed_kernel<SwT, MobT, IN64, MOBIN>), lds,
                  lds_wgs(lds, sizeof(SwT) == 4 ? 2 : 1)};
}
template <bool MOBIN>
static FastForm form_m(int prec, int l, int np) {
  switch (prec) {
    case PREC_F32: return form_t<float, float, false, MOBIN>(l, np);
    case PREC_F32_COMP: return form_t<float, TwoF, false, MOBIN>(l, np);
    case PREC_F64: return form_t<double, double, true, MOBIN>(l, np);
    default: return form_t<float, double, false, MOBIN>(l, np);
  }
}
// l = 0: the kernel over every order. Plans whose input is already the Moebius
// transform run their own instantiations.
static FastForm fast_form(int prec, int l, int np, int mobius_in) {
  return mobius_in ? form_m<true>(prec, l, np) : form_m<false>(prec, l, np);
}

// LDS bytes of a launch: the form's, or more where the grid is smaller than the
// machine holds, so that no CU takes more workgroups than an even spread gives
// it (the dispatcher otherwise fills a CU before it goes to the next one: 500 x
// d = 14, l = 3 in FP32 54 us on 167 CUs, 34 spread over all). Not for a grid of at
// most one workgroup per CU: the dispatcher spreads it by itself (single d = 20,
// l = 4 in FP32 19.3 us with and without), and the launches of other streams find
// room beside it (two streams of them 17.5 us an apply with, 12.0 without).
static unsigned spread_lds(const FastForm& form, int grid, int n_cu) {
  const int share = (grid + n_cu - 1) / n_cu;
  if (share == 1 || share >= form.wgs) return (unsigned)form.lds;
  return (unsigned)std::max(form.lds, 160 * 1024 / share - 2048);
}

static hipError_t launch_items(const FastLaunch& f, int l, int ib, int n, int grid, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const FastForm form = fast_form(f.prec, l, f.np[l], f.mobius_in);
  const FastItem* items = f.items + ib;
  const float* v32 = static_cast<const float*>(f.vals32);
  const double* v64 = static_cast<const double*>(f.vals64);
  void* out = f.out;
  void* args[] = {(void*)&f.classes, (void*)&f.insts, (void*)&items, (void*)&n, (void*)&v32,
                  (void*)&v64, (void*)&f.torder, (void*)&f.partial, (void*)&out, (void*)&f.queue};
  return hipLaunchKernel(form.fn, dim3(grid), dim3(NT), args, spread_lds(form, grid, f.n_cu), st);
}

hipError_t launch_fast_mixed(const FastLaunch& f, hipStream_t st) {
  return launch_items(f, 0, 0, f.n_items, f.grid_mixed, st);
}

hipError_t launch_fast_group(const FastLaunch& f, int l, hipStream_t st) {
  return launch_items(f, l, f.lbeg[l], f.lbeg[l + 1] - f.lbeg[l], f.grid[l], st);
}

hipError_t configure_fast(int prec, const int* np) {
  int orders = 0;
  for (int l = 1; l <= kFastMaxL; ++l) orders += np[l] > 0;
  for (int l = orders > 1 ? 0 : 1; l <= kFastMaxL; ++l) {
    if (l > 0 && np[l] == 0) continue;
    for (int m = 0; m < 2; ++m) {
      const FastForm form = fast_form(prec, l, np[l], m);
      const hipError_t e =
          hipFuncSetAttribute(form.fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              std::max(form.lds, 160 * 1024 - 2048));
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

int fast_groups(const FastLaunch& f, int* ls) {
  int n = 0;
  for (int l = 1; l <= kFastMaxL; ++l)
    if (f.lbeg[l + 1] > f.lbeg[l]) {
      if (ls) ls[n] = l;
      ++n;
    }
  return n;
}

int fast_launches(const FastLaunch& f) {
  const int g = fast_groups(f, nullptr);
  return g > 1 ? 1 : g;
}

bool fast_supported(int prec) {
  return prec == PREC_F32 || prec == PREC_F32_COMP || prec == PREC_F32_FP64MOB ||
         prec == PREC_F64;
}

// Workgroups of the kernel of order l (0: of every order) that fit on one CU.
int fast_wgs_per_cu(int prec, int l, int np) { return fast_form(prec, l, np, 0).wgs; }

}  // namespace fsi
