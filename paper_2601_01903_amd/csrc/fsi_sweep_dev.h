// Device code of the register-phase counter sweep (tiles of 2^11 values),
// shared by the kernel of orders l <= 4 (fsi_tile11.hip) and the kernel of
// orders 5 and 6 (fsi_tile_high.hip): numerics of the butterfly forms, the
// in-register sweep, the emitters of its three phases and phases B and C.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "fsi_tile11.h"

namespace fsi {
namespace t11 {

// ----------------------------------------------------------------- numerics
struct TwoF {
  float hi, lo;
};
// Two-float subtraction: Knuth's TwoSum of the high parts (exact error e),
// the low parts and e added into the low word. The pair is not renormalised
// (hi + lo still holds the value; the low word stays within a few ulps of the
// operands over the 11 butterfly levels) and is rounded once, to FP32, when
// the sweep takes it.
__device__ __forceinline__ TwoF sub(TwoF a, TwoF b) {
  const float s = a.hi - b.hi;
  const float bb = s - a.hi;
  const float e = (a.hi - (s - bb)) + (-b.hi - bb);
  return TwoF{s, e + (a.lo - b.lo)};
}
// The same, renormalised after every level (orders 5 and 6, as on the generic
// kernel): the low word stays within half an ulp of the high one and so keeps
// its own last bits. Values up to 1.5e7 that cancel, beside values of 0.025: rms
// error of a coefficient 1.7e-9 renormalised, 2.5e-9 not; 1 to 3% of the time.
struct TwoFN {
  float hi, lo;
};
__device__ __forceinline__ TwoFN sub(TwoFN a, TwoFN b) {
  const TwoF x = sub(TwoF{a.hi, a.lo}, TwoF{b.hi, b.lo});
  const float hi = x.hi + x.lo;
  return TwoFN{hi, x.lo - (hi - x.hi)};
}
__device__ __forceinline__ float sub(float a, float b) { return a - b; }
__device__ __forceinline__ double sub(double a, double b) { return a - b; }

template <typename M> __device__ __forceinline__ M mob_from(float x);
template <> __device__ __forceinline__ float mob_from<float>(float x) { return x; }
template <> __device__ __forceinline__ double mob_from<double>(float x) { return x; }
template <> __device__ __forceinline__ TwoF mob_from<TwoF>(float x) { return TwoF{x, 0.f}; }
template <> __device__ __forceinline__ TwoFN mob_from<TwoFN>(float x) { return TwoFN{x, 0.f}; }
template <typename M> __device__ __forceinline__ M mob_from_d(double x);
template <> __device__ __forceinline__ double mob_from_d<double>(double x) { return x; }

template <typename S> __device__ __forceinline__ S to_sw(float x) { return (S)x; }
template <typename S> __device__ __forceinline__ S to_sw(double x) { return (S)x; }
template <typename S> __device__ __forceinline__ S to_sw(TwoF x);
template <> __device__ __forceinline__ float to_sw<float>(TwoF x) { return x.hi + x.lo; }
template <typename S> __device__ __forceinline__ S to_sw(TwoFN x) { return to_sw<S>(TwoF{x.hi, x.lo}); }
template <> __device__ __forceinline__ double to_sw<double>(TwoF x) {
  return (double)x.hi + (double)x.lo;
}

// ------------------------------------------------- in-register counter sweep
// Node of the depth-first walk over the output bits of one phase: X[t][r]
// holds the states with counter t in [LO, LO + RC) for the 2^REM inputs r of
// the bits still to consume. The most significant remaining bit is consumed
// first: the sigma = 1 child keeps the tau = 1 half with t + 1; the sigma = 0
// child adds the tau = 0 half at t and the tau = 1 half at t - 1. At a leaf
// SIG is the output mask over the phase's bits and X[i] holds counter LO + i,
// i.e. the counter relative to the prefix's popcount (LO = |SIG|).
template <int REM, int LO, int RC, int SIG, typename T, typename Emit>
__device__ __forceinline__ void rsweep(const T (&X)[RC][1 << REM], Emit& emit) {
  if constexpr (REM == 0) {
    emit.template leaf<SIG, LO, RC>(X);
  } else {
    constexpr int H = 1 << (REM - 1);
    {
      T Y0[RC + 1][H];
#pragma unroll
      for (int r = 0; r < H; ++r) {
        Y0[0][r] = X[0][r];
#pragma unroll
        for (int t = 1; t < RC; ++t) Y0[t][r] = X[t][r] + X[t - 1][H + r];
        Y0[RC][r] = X[RC - 1][H + r];
      }
      rsweep<REM - 1, LO, RC + 1, SIG>(Y0, emit);
    }
    {
      T Y1[RC][H];
#pragma unroll
      for (int t = 0; t < RC; ++t)
#pragma unroll
        for (int r = 0; r < H; ++r) Y1[t][r] = X[t][H + r];
      rsweep<REM - 1, LO + 1, RC, SIG | H>(Y1, emit);
    }
  }
}

// Raw-tile transposes: element (a, b, c) of the tile (index a + 16 b + 256 c)
// at a + 17 b + 272 c. Affine in each coordinate, so every access is a
// per-thread base plus an immediate; the three access patterns (fixed c,
// fixed b, fixed a across a wave) hit distinct banks (fixed c: 3 of 64
// banks shared).
constexpr int RB = 17, RC_ = 272;
constexpr int r_elems = RC_ * NC;

// Weights are read-only for the whole launch: addressed through the constant
// address space, so wave-uniform reads become scalar loads.
typedef const __attribute__((address_space(4))) double* cdptr;
typedef const __attribute__((address_space(4))) uint32_t* cdptr_u;

template <typename T> struct Vec4;
template <> struct Vec4<float> { using type = float4; static constexpr int n = 4; };
template <> struct Vec4<double> { using type = double2; static constexpr int n = 2; };

// Compile-time tables of one order l (indexed with unrolled loop counters,
// so every use folds into an immediate).
struct A5 { int v[PA + 1]; };
struct A16 { int v[16]; };
constexpr A5 mk_off1(int L) {
  A5 a{};
  for (int r = 0; r <= PA; ++r) a.v[r] = off1(L, r);
  return a;
}
constexpr A16 mk_ubase(int L) {
  A16 a{};
  for (int b = 0; b < NB; ++b) a.v[b] = ubase(L, b);
  return a;
}
constexpr A16 mk_rank() {
  A16 a{};
  for (int m = 0; m < NA; ++m) a.v[m] = rankA(m);
  return a;
}
template <int L>
struct K {
  static constexpr A5 off1v = mk_off1(L);
  static constexpr A16 ub = mk_ubase(L);
  static constexpr A16 rk = mk_rank();
  static constexpr int N3 = n3(L);
  static constexpr int S2U = s2u(L);
  static constexpr int LB = lamblock(L);
  static constexpr int NTASK = ntasks(L);
  static constexpr int NPAIR = npairs(L);
  static constexpr int LAM0 = lamoff(L, 0), LAM1 = lamoff(L, 1);
  static constexpr int YB0 = ybase(L, 0), YB1 = ybase(L, 1);
};

// ----------------------------------------------------------------- emitters
// Phase A -> S1 row off1(i) + rankA(sigma_A), column = this thread's input.
template <typename SwT, int L>
struct EmitS1 {
  SwT* S1;   // already offset by the thread's column
  template <int SIG, int LO, int RC>
  __device__ __forceinline__ void leaf(const SwT (&X)[RC][1]) {
    if constexpr (cpop(SIG) <= L) {
      constexpr int R1 = row1_stride<SwT>();
      constexpr int RK = K<L>::rk.v[SIG];
#pragma unroll
      for (int i = 0; i < RC; ++i) S1[(K<L>::off1v.v[i] + RK) * R1] = X[i][0];
    }
  }
};

// Phase B -> S2 entries (i, unit of (sigma_A, sigma_B), c) for the leaf's
// counters i < RC (entries past this unit's range hold zeros), for the
// prefixes with |sigma_A| + |sigma_B| <= L. Phase C reads only i <= 8 - |sigma_AB|,
// all written here.
template <typename SwT, int L, int SAMIN, int SAMAX>
struct EmitS2 {
  SwT* S2;   // offset by ((c / 4) * s2u + rankA) * 4 + c % 4
  int sA;    // in [SAMIN, SAMAX]
  int rkA;   // rankA
  template <int SIG, int LO, int RC>
  __device__ __forceinline__ void leaf(const SwT (&X)[RC][1]) {
    constexpr int sB = cpop(SIG);
    if constexpr (sB <= L - SAMIN) {
      constexpr int UB = K<L>::ub.v[SIG];
      constexpr int S2U = K<L>::S2U;
      if constexpr (sB <= L - SAMAX) {
#pragma unroll
        for (int i = 0; i < RC; ++i) S2[(2 * i * S2U + UB) * 4] = X[i][0];
      } else {
        // a prefix past the order writes a padding unit (n3 .. s2u - 1),
        // which phase C never reads
        const int ub = sA <= L - sB ? UB : K<L>::N3 - rkA;
#pragma unroll
        for (int i = 0; i < RC; ++i) S2[(2 * i * S2U + ub) * 4] = X[i][0];
      }
    }
  }
};

// Phase C -> Z row of S_L = sigma_AB | sigma_C << 8 (12 entries, zero padded).
template <typename SwT, int L, int KMIN, int KMAX>
struct EmitZ {
  SwT* Z;
  const int (&zr)[NC];   // Z row per sigma_C (dump row where |S_L| > L)
  int sAB;               // in [KMIN, KMAX] for every unit of the wave
  template <int SIG, int LO, int RC>
  __device__ __forceinline__ void leaf(const SwT (&X)[RC][1]) {
    constexpr int sC = cpop(SIG);
    if constexpr (sC <= L - KMIN) {
      {   // leaves past the order write the dump row (zr)
        using V = typename Vec4<SwT>::type;
        constexpr int VN = Vec4<SwT>::n;
        V* p = reinterpret_cast<V*>(Z + zr[SIG] * ZROW);
        // the weight core reads a row's counters only (the first 12 - |S_L|
        // entries, at most RC here): the padding past them is not stored
#pragma unroll
        for (int q = 0; q < (RC + VN - 1) / VN; ++q) {
          SwT e[VN];
#pragma unroll
          for (int k = 0; k < VN; ++k) e[k] = q * VN + k < RC ? X[q * VN + k][0] : SwT(0);
          if constexpr (VN == 4) p[q] = V{e[0], e[1], e[2], e[3]};
          else p[q] = V{e[0], e[1]};
        }
      }
    }
  }
};

// Phase B of one wave: every sigma_A of the wave has SAMIN <= |sigma_A| <=
// SAMAX, so its counter rows past PA - SAMIN are zero and its leaves with
// |sigma_B| > L - SAMIN are never written (both dropped at compile time),
// while rows up to PA - SAMAX and leaves with |sigma_B| <= L - SAMAX need no
// run-time test. HALF 0 walks the sigma = 0 subtree of the first output site
// (all 16 inputs), HALF 1 the sigma = 1 subtree (the 8 tau = 1 inputs). BAR:
// S2 overlays S1, so every wave has its inputs in registers before one stores.
constexpr int kSALoMax = cpop(orderA(7));   // |sigma_A| of rank 7
constexpr int kSAHi = cpop(orderA(8));      // |sigma_A| of rank 8
constexpr int kSAHiMax = cpop(orderA(15));  // |sigma_A| of rank 15
template <int L, int SAMIN, int SAMAX, int HALF, typename SwT, bool BAR = false>
__device__ __forceinline__ void phase_b(const SwT* S1, SwT* S2w, int sA, int p2r, int p2c) {
  if constexpr (SAMIN <= L) {
    const bool off = SAMAX > L && sA > L;   // nothing to write
    if (!BAR && off) return;
    using V = typename Vec4<SwT>::type;
    constexpr int VN = Vec4<SwT>::n;
    constexpr int H = NB / 2;
    constexpr int R1 = row1_stride<SwT>();
    constexpr int NRB = PA + 1 - SAMIN;
    constexpr int W = HALF == 0 ? NB : H;       // inputs this half reads
    EmitS2<SwT, L, SAMIN, SAMAX> e2{S2w, sA, p2r};
    const SwT* src0 = S1 + p2r * R1 + NB * p2c + (HALF == 0 ? 0 : H);
    SwT X[NRB][W];
#pragma unroll
    for (int r = 0; r < NRB; ++r) {
      if (r <= PA - SAMAX || r <= PA - sA) {
        const V* src = reinterpret_cast<const V*>(src0 + K<L>::off1v.v[r] * R1);
#pragma unroll
        for (int q = 0; q < W / VN; ++q) {
          const V v = src[q];
          if constexpr (VN == 4) {
            X[r][4 * q] = v.x; X[r][4 * q + 1] = v.y; X[r][4 * q + 2] = v.z; X[r][4 * q + 3] = v.w;
          } else {
            X[r][2 * q] = v.x; X[r][2 * q + 1] = v.y;
          }
        }
      } else {
#pragma unroll
        for (int b = 0; b < W; ++b) X[r][b] = SwT(0);
      }
    }
    if constexpr (BAR) __syncthreads();
    if (BAR && off) return;
    if constexpr (HALF == 0) {
      SwT Y0[NRB + 1][H];
#pragma unroll
      for (int j = 0; j < H; ++j) {
        Y0[0][j] = X[0][j];
#pragma unroll
        for (int t = 1; t < NRB; ++t) Y0[t][j] = X[t][j] + X[t - 1][H + j];
        Y0[NRB][j] = X[NRB - 1][H + j];
      }
      rsweep<PB - 1, 0, NRB + 1, 0>(Y0, e2);
    } else {
      rsweep<PB - 1, 1, NRB, H>(X, e2);
    }
  }
}

template <int L> struct UO { static constexpr UnitOrder o = mk_unit_order(L); };

// Phase C of one wave: its units have KMIN <= |sigma_AB| <= KMAX. Counter
// rows past KAB - |sigma_AB| are zero: dropped at compile time past
// KAB - KMIN, and below that read as zeros (a zeroed LDS row where KMIN = 0,
// so the loads issue without branches). PART 2 walks all output prefixes over
// the C bits; PART 0 the sigma = 0 subtree of the first C site (all 8
// inputs), PART 1 its sigma = 1 subtree (the 4 tau = 1 inputs).
template <int L, int KMIN, int KMAX, int PART, typename SwT, bool BAR = false>
__device__ __forceinline__ void phase_c(const SwT* S2, SwT* Z, const int (&zr)[NC], int sAB,
                                        int u3, const SwT* zrow) {
  if constexpr (KMIN <= L) {
    using V = typename Vec4<SwT>::type;
    constexpr int VN = Vec4<SwT>::n;
    constexpr int S2U = K<L>::S2U;
    constexpr int NR = KAB + 1 - KMIN;
    constexpr int H0 = PART == 1 ? 1 : 0;       // first half (c / 4) read
    constexpr int W = PART == 1 ? NC / 2 : NC;  // inputs read
    SwT X3[NR][W];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const bool in = i <= KAB - KMAX || i <= KAB - sAB;
      if (KMIN > 0 && !in) {   // past this unit's counters: zero, not read
#pragma unroll
        for (int c = 0; c < W; ++c) X3[i][c] = SwT(0);
        continue;
      }
#pragma unroll
      for (int h = H0; h < 2; ++h) {
        const V* src = reinterpret_cast<const V*>(
            KMIN > 0 || in ? S2 + ((2 * i + h) * S2U + u3) * 4 : zrow);
#pragma unroll
        for (int q = 0; q < 4 / VN; ++q) {
          const V v = src[q];
          const int c0 = 4 * (h - H0) + VN * q;
          if constexpr (VN == 4) {
            X3[i][c0] = v.x; X3[i][c0 + 1] = v.y; X3[i][c0 + 2] = v.z; X3[i][c0 + 3] = v.w;
          } else {
            X3[i][c0] = v.x; X3[i][c0 + 1] = v.y;
          }
        }
      }
    }
    if constexpr (BAR) __syncthreads();   // Z overlays S2
    EmitZ<SwT, L, KMIN, KMAX> ez{Z, zr, sAB};
    if constexpr (PART == 2) {
      rsweep<PC, 0, NR, 0>(X3, ez);
    } else if constexpr (PART == 0) {
      constexpr int H = NC / 2;
      SwT Y0[NR + 1][H];
#pragma unroll
      for (int j = 0; j < H; ++j) {
        Y0[0][j] = X3[0][j];
#pragma unroll
        for (int t = 1; t < NR; ++t) Y0[t][j] = X3[t][j] + X3[t - 1][H + j];
        Y0[NR][j] = X3[NR - 1][H + j];
      }
      rsweep<PC - 1, 0, NR + 1, 0>(Y0, ez);
    } else {
      rsweep<PC - 1, 1, NR, NC / 2>(X3, ez);
    }
  }
}

}  // namespace t11
}  // namespace fsi
