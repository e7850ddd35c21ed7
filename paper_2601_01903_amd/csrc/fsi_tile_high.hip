// Register-phase tile kernel of orders 5 and 6 (fused algorithm, gfx950).
//
// The in-tile work is that of the kernel of orders l <= 4 (fsi_tile11.hip):
// the butterfly over 11 low bits, then the counter sweep in register phases
// of 4, 4 and 3 sites (fsi_sweep_dev.h). The differences follow from the
// number of outputs: they outnumber a workgroup's accumulators (21,700 at
// d = 20, l = 5), so the per-tile results Y go to memory and a reduction adds
// them over the tiles; and the sweep states outgrow the regions, so the
// phases share one: each reads its inputs into registers, a barrier, then
// stores over them. That leaves two workgroups per CU in FP32 (64 and 72 KB
// at l = 5, 6), one in FP64.
//
// Bound: LDS traffic of the states. The generic kernel it replaces for these
// orders held one state per thread and LDS round trip and site; measured on
// 8 instances of d = 18, l = 6 (FP32, FP64 butterfly): tile kernel 238 us and
// reduction 95 us, here 25 us and 32 us.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "fsi_kernels.h"
#include "fsi_sweep_dev.h"
#include "fsi_tile11.h"

namespace fsi {
namespace t11 {

constexpr int imaxh(int a, int b) { return a > b ? a : b; }
template <int L, typename SwT, typename MobT>
struct LdsHigh {
  // the transposes at 0, the phase-A states S1 after them; S2 over both; Z
  // over S2
  static constexpr int s1off = (int)((r_elems * sizeof(MobT) + 255) & ~255);
  static constexpr int s1end = s1off + rows1(L) * row1_stride<SwT>() * (int)sizeof(SwT);
  static constexpr int s2 = s2_elems(L) * (int)sizeof(SwT);
  static constexpr int z = (nzrows(L) + 1) * ZROW * (int)sizeof(SwT);
  static constexpr int zoff = (imaxh(s1end, imaxh(s2, z)) + 255) & ~255;   // zero row
  static constexpr int bytes = zoff + 128;
  static_assert(bytes <= 160 * 1024, "LDS");
};

// ---- final weights: 64-lane tasks, as in the kernel of orders l <= 4 (rows
// of one |S_L| >= 2 with uniform weights, slots [k0, k1) of each; (row, slot)
// pairs of |S_L| <= 1 with per-lane weights), dealt to the waves longest
// first. Each result goes straight to Y in memory, coalesced over the rows.
struct HighTask { int pair, S, chunk, k0, k1, cost, wave; };
struct HighPlan { HighTask t[80]; int n; };
constexpr int kHighSlots = 8;   // slots of a task: accumulators per lane
constexpr HighPlan make_high_plan(int L) {
  HighPlan p{};
  for (int S = L; S >= 2; --S) {
    const int NS = nslots(L, S), parts = (NS + kHighSlots - 1) / kHighSlots;
    for (int c = 0; c < row_tasks(S); ++c)
      for (int q = 0; q < parts; ++q) {
        const int k0 = NS * q / parts, k1 = NS * (q + 1) / parts;
        p.t[p.n++] = HighTask{0, S, c, k0, k1, (k1 - k0 + 2) * (ZROW - S) + 8, -1};
      }
  }
  for (int c = 0; c < (npairs(L) + 63) / 64; ++c)
    p.t[p.n++] = HighTask{1, 0, c, 0, 0, 4 * ZROW + 8, -1};
  int load[NT / 64] = {};
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
template <int L> struct HP { static constexpr HighPlan plan = make_high_plan(L); };

template <int N, typename SwT>
__device__ __forceinline__ void load_row(const SwT* zr, double (&z)[N]) {
  using V = typename Vec4<SwT>::type;
  constexpr int VN = Vec4<SwT>::n;
  const V* zv = reinterpret_cast<const V*>(zr);
#pragma unroll
  for (int q = 0; q < (N + VN - 1) / VN; ++q) {
    const V v = zv[q];
    SwT e[VN];
    if constexpr (VN == 4) { e[0] = v.x; e[1] = v.y; e[2] = v.z; e[3] = v.w; }
    else { e[0] = v.x; e[1] = v.y; }
#pragma unroll
    for (int k = 0; k < VN; ++k)
      if (q * VN + k < N) z[q * VN + k] = (double)e[k];
  }
}

// h: high bits of the instance (slots of s_H > h do not exist)
template <int L, int W, int J, typename SwT>
__device__ __forceinline__ void high_tasks(int lane, int h, const SwT* Z, const double* lam, cdptr lamg,
                                           double* __restrict__ Y) {
  if constexpr (J < HP<L>::plan.n) {
    constexpr HighTask T = HP<L>::plan.t[J];
    if constexpr (T.wave == W) {
      if constexpr (!T.pair) {
        constexpr int S = T.S, K0 = T.k0, K1 = T.k1, RC = ZROW - S, NR = cbinom(B, S);
        constexpr int LO = lamoff(L, S), YB = ybase(L, S);
        const int top = min(L - S, h), ns = (top + 1) * (top + 2) / 2;
        if (K0 < ns) {
          const int row = T.chunk * 64 + lane;
          const bool ok = (T.chunk + 1) * 64 <= NR || row < NR;
          double z[RC];
          load_row<RC, SwT>(Z + (zbase(S) + (ok ? row : 0)) * ZROW, z);
          double a[K1 - K0];
#pragma unroll
          for (int k = K0; k < K1; ++k) a[k - K0] = 0.0;
#pragma unroll
          for (int r = 0; r < RC; ++r)
#pragma unroll
            for (int k = K0; k < K1; ++k) a[k - K0] = fma(lamg[LO + k * ZROW + r], z[r], a[k - K0]);
          if (ok) {
#pragma unroll
            for (int k = K0; k < K1; ++k)
              if (k < ns) Y[YB + k * nrp(S) + row] = a[k - K0];
          }
        }
      } else {
        constexpr int N0 = nslots(L, 0), N1 = nslots(L, 1);
        const int p = T.chunk * 64 + lane;
        if (p < npairs(L)) {
          const bool z0 = p < N0;
          const int row = z0 ? 0 : (p - N0) / N1, slot = z0 ? p : (p - N0) - row * N1;
          const int top = min(z0 ? L : L - 1, h);
          if (slot < (top + 1) * (top + 2) / 2) {
            double z[ZROW];
            load_row<ZROW, SwT>(Z + (z0 ? 0 : 1 + row) * ZROW, z);
            // entry 11 of an |S_L| = 1 row lies past its counters
            if (!z0) z[ZROW - 1] = 0.0;
            const double2* lw = reinterpret_cast<const double2*>(
                lam + (z0 ? lamoff(L, 0) : lamoff(L, 1)) + slot * ZROW);
            double a = 0.0;
#pragma unroll
            for (int q = 0; q < ZROW / 2; ++q) {
              const double2 w = lw[q];
              a = fma(w.x, z[2 * q], a);
              a = fma(w.y, z[2 * q + 1], a);
            }
            Y[z0 ? ybase(L, 0) + slot * nrp(0) : ybase(L, 1) + slot * nrp(1) + row] = a;
          }
        }
      }
    }
    high_tasks<L, W, J + 1, SwT>(lane, h, Z, lam, lamg, Y);
  }
}

template <int L, typename SwT, typename MobT, bool IN64, int WPE, bool MOBIN>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE)))
tile_high_kernel(const FastClassDev* __restrict__ classes, const InstDev* __restrict__ insts,
                 const TileItem* __restrict__ items, int n_items,
                 const typename std::conditional<IN64, double, float>::type* __restrict__ vals,
                 double* __restrict__ Yall) {
  extern __shared__ __align__(16) unsigned char smem[];
  using LD = LdsHigh<L, SwT, MobT>;
  using RawT = typename std::conditional<IN64, double, float>::type;
  MobT* R = reinterpret_cast<MobT*>(smem);
  SwT* S1 = reinterpret_cast<SwT*>(smem + LD::s1off);
  SwT* S2 = reinterpret_cast<SwT*>(smem);
  SwT* Z = reinterpret_cast<SwT*>(smem);
  SwT* zrow = reinterpret_cast<SwT*>(smem + LD::zoff);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < 128 / 4) reinterpret_cast<uint32_t*>(zrow)[tid] = 0u;

  const int p2r = (((tid & 127) >> 6) << 3) | (tid & 7), p2c = (tid >> 3) & 7;
  const int sA = __popc((unsigned)((kOrderANibbles >> (4 * p2r)) & 15u));
  const int wb = ((p2c >> 2) * K<L>::S2U + p2r) * 4 + (p2c & 3);

  RawT xraw[NC];
  auto load_tile = [&](const TileItem& w) {
    const InstDev& I = insts[w.inst];
    const int lowmask = I.lowmask;
    const RawT* v = vals + I.voff + ((int64_t)w.tile << B);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int idx = tid + (c << 8);
      // d < 11: the value of U is v(U & lowmask); Moebius coefficients past
      // bit d - 1 are zero
      if constexpr (MOBIN) xraw[c] = idx <= lowmask ? v[idx & lowmask] : RawT(0);
      else xraw[c] = v[idx & lowmask];
    }
  };
  int it = blockIdx.x;
  if (it < n_items) load_tile(items[it]);
  for (; it < n_items; it += gridDim.x) {
    const TileItem w = items[it];
    const InstDev& I = insts[w.inst];
    const FastClassDev* C = classes + I.fcls;
    // ---- butterfly over bits 8-10 in registers, then 4-7 ----
    {
      MobT xr[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if constexpr (IN64) xr[c] = mob_from_d<MobT>(xraw[c]);
        else xr[c] = mob_from<MobT>(xraw[c]);
      }
      if constexpr (!MOBIN) {
#pragma unroll
        for (int bit = 0; bit < PC; ++bit)
#pragma unroll
          for (int c = 0; c < NC; ++c)
            if (c & (1 << bit)) xr[c] = sub(xr[c], xr[c ^ (1 << bit)]);
      }
      MobT* rp = R + (tid & 15) + RB * (tid >> 4);
#pragma unroll
      for (int c = 0; c < NC; ++c) rp[RC_ * c] = xr[c];
    }
    __syncthreads();
    if (!MOBIN && tid < NA * NC) {
      MobT* rp = R + (tid & 15) + RC_ * (tid >> 4);
      MobT y[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) y[b] = rp[RB * b];
#pragma unroll
      for (int bit = 0; bit < PB; ++bit)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (b & (1 << bit)) y[b] = sub(y[b], y[b ^ (1 << bit)]);
#pragma unroll
      for (int b = 0; b < NB; ++b) rp[RB * b] = y[b];
    }
    __syncthreads();
    // ---- bits 0-3 and phase A ----
    if (tid >= NT - NB * NC) {
      const int ta = tid - (NT - NB * NC);
      const MobT* rp = R + RB * (ta & 15) + RC_ * (ta >> 4);
      MobT y[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) y[a] = rp[a];
      if constexpr (!MOBIN) {
#pragma unroll
        for (int bit = 0; bit < PA; ++bit)
#pragma unroll
          for (int a = 0; a < NA; ++a)
            if (a & (1 << bit)) y[a] = sub(y[a], y[a ^ (1 << bit)]);
      }
      SwT X1[1][NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) X1[0][a] = to_sw<SwT>(y[a]);
      // d < 11: the coefficients past bit d - 1 are differences of equal
      // values, zero unless those are infinite
      const int lowmask = I.lowmask;
      if (!MOBIN && lowmask < (1 << B) - 1) {
#pragma unroll
        for (int a = 0; a < NA; ++a)
          if ((ta << PA | a) > lowmask) X1[0][a] = SwT(0);
      }
      EmitS1<SwT, L> e1{S1 + ta};
      rsweep<PA, 0, 1, 0>(X1, e1);
    }
    __syncthreads();
    // ---- phase B (its barrier: S2 overlays S1) ----
    switch (wave) {
      case 0: phase_b<L, 0, kSALoMax, 0, SwT, true>(S1, S2 + wb, sA, p2r, p2c); break;
      case 1: phase_b<L, kSAHi, kSAHiMax, 0, SwT, true>(S1, S2 + wb, sA, p2r, p2c); break;
      case 2: phase_b<L, 0, kSALoMax, 1, SwT, true>(S1, S2 + wb, sA, p2r, p2c); break;
      default: phase_b<L, kSAHi, kSAHiMax, 1, SwT, true>(S1, S2 + wb, sA, p2r, p2c); break;
    }
    __syncthreads();
    // ---- phase C (its barrier: Z overlays S2): a unit per thread; threads
    // past the units run unit 0 into the dump row ----
    {
      const int ur = C->uperm[tid];
      const int u3 = ur >= 0 ? ur : 0;
      using O = UO<L>;
      const int sAB = ur >= 0 ? __popc((unsigned)C->unit_mask[u3]) : O::o.kmax[NT / 64 - 1];
      int zr[NC];
#pragma unroll
      for (int sc = 0; sc < NC; ++sc) zr[sc] = ur >= 0 ? C->zrow[u3 * NC + sc] : nzrows(L);
      switch (wave) {
        case 0: phase_c<L, O::o.kmin[0], O::o.kmax[0], 2, SwT, true>(S2, Z, zr, sAB, u3, zrow); break;
        case 1: phase_c<L, O::o.kmin[1], O::o.kmax[1], 2, SwT, true>(S2, Z, zr, sAB, u3, zrow); break;
        case 2: phase_c<L, O::o.kmin[2], O::o.kmax[2], 2, SwT, true>(S2, Z, zr, sAB, u3, zrow); break;
        default: phase_c<L, O::o.kmin[3], O::o.kmax[3], 2, SwT, true>(S2, Z, zr, sAB, u3, zrow); break;
      }
    }
    if (it + (int)gridDim.x < n_items) load_tile(items[it + gridDim.x]);
    __syncthreads();
    // ---- final weights -> Y ----
    {
      const int u = __builtin_amdgcn_readfirstlane(__popc((unsigned)w.tile));
      const double* lam = C->lam + (int64_t)u * K<L>::LB;
      const cdptr lamg = (cdptr)lam;
      double* Y = Yall + I.yoff + (int64_t)w.tile * ysize(L);
      const int h = C->h;
      switch (wave) {
        case 0: high_tasks<L, 0, 0, SwT>(lane, h, Z, lam, lamg, Y); break;
        case 1: high_tasks<L, 1, 0, SwT>(lane, h, Z, lam, lamg, Y); break;
        case 2: high_tasks<L, 2, 0, SwT>(lane, h, Z, lam, lamg, Y); break;
        default: high_tasks<L, 3, 0, SwT>(lane, h, Z, lam, lamg, Y); break;
      }
    }
    __syncthreads();
  }
}

// Sum over the tiles: output k of an instance takes, from tile U, entry
// base + |S_H & U| * stride of its per-tile results (base and stride packed
// in hword). A workgroup owns 256 / ROWS consecutive outputs; row r adds the
// tiles U = r mod ROWS in increasing order, then the rows are added in order.
// Moebius input (inside = ~0, else 0): only the tiles with S_H inside U hold
// coefficients of supersets; the others' entries are sums of zero weights, NaN
// where a coefficient is infinite.
template <typename OutT, int ROWS>
__global__ void __launch_bounds__(NT)
high_reduce_kernel(const InstDev* __restrict__ insts, const int2* __restrict__ chunks, int n_chunks,
                   uint32_t inside, const double* __restrict__ Yall, OutT* __restrict__ out) {
  constexpr int W = NT / ROWS;
  __shared__ double part[ROWS][W];
  const int o = threadIdx.x % W, r = threadIdx.x / W;
  for (int ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
    const int2 c = chunks[ch];
    const InstDev& I = insts[c.x];
    const int k = c.y + o;
    double acc = 0.0;
    if (k < I.nout) {
      const uint32_t word = I.hword[k], SH = I.hhigh[k];
      const uint32_t stride = word >> 16;
      const double* Y = Yall + I.yoff + (word & 0xffffu);
      const uint32_t nt = 1u << I.nhigh;
#pragma unroll 8
      for (uint32_t U = r; U < nt; U += ROWS) {
        const double y = Y[(int64_t)U * I.pstride + __popc(SH & U) * stride];
        acc += (SH & ~U & inside) ? 0.0 : y;
      }
    }
    if constexpr (ROWS > 1) {
      part[r][o] = acc;
      __syncthreads();
      if (r == 0)
#pragma unroll
        for (int q = 1; q < ROWS; ++q) acc += part[q][o];
      __syncthreads();
    }
    if (r == 0 && k < I.nout) out[I.ooff + k] = (OutT)acc;
  }
}

template <typename SwT> constexpr int wpe_high() { return sizeof(SwT) == 4 ? 2 : 1; }

}  // namespace t11

using namespace t11;

template <int L, typename SwT, typename MobT, bool IN64, bool MOBIN>
static hipError_t launch_high_m(const HighLaunch& f, const void* vals, double* Y, hipStream_t st) {
  using RawT = typename std::conditional<IN64, double, float>::type;
  const int ib = f.lbeg[L - kHighMinL], n = f.lbeg[L - kHighMinL + 1] - ib;
  if (n <= 0) return hipSuccess;
  auto k = tile_high_kernel<L, SwT, MobT, IN64, wpe_high<SwT>(), MOBIN>;
  constexpr int lds = LdsHigh<L, SwT, MobT>::bytes;
  const int grid = std::min(n, f.n_cu * std::max(1, 160 * 1024 / lds));
  hipLaunchKernelGGL(k, dim3(grid), dim3(NT), lds, st, f.classes, f.insts, f.items + ib, n,
                     static_cast<const RawT*>(vals), Y);
  return hipGetLastError();
}
template <int L, typename SwT, typename MobT, bool IN64>
static hipError_t launch_high_l(const HighLaunch& f, const void* vals, double* Y, hipStream_t st) {
  return f.mobius_in ? launch_high_m<L, SwT, MobT, IN64, true>(f, vals, Y, st)
                     : launch_high_m<L, SwT, MobT, IN64, false>(f, vals, Y, st);
}
template <typename SwT, typename MobT, bool IN64>
static hipError_t launch_high_t(const HighLaunch& f, int l, const void* vals, double* Y, hipStream_t st) {
  return l == 5 ? launch_high_l<5, SwT, MobT, IN64>(f, vals, Y, st)
                : launch_high_l<6, SwT, MobT, IN64>(f, vals, Y, st);
}

hipError_t launch_high(const HighLaunch& f, int l, const void* vals, double* Y, hipStream_t st) {
  switch (f.prec) {
    case PREC_F32: return launch_high_t<float, float, false>(f, l, vals, Y, st);
    case PREC_F32_COMP: return launch_high_t<float, TwoFN, false>(f, l, vals, Y, st);
    case PREC_F32_FP64MOB: return launch_high_t<float, double, false>(f, l, vals, Y, st);
    case PREC_F64: return launch_high_t<double, double, true>(f, l, vals, Y, st);
  }
  return hipErrorInvalidValue;
}

template <typename OutT>
static hipError_t launch_high_reduce_t(const HighLaunch& f, const double* Y, void* out, hipStream_t st) {
  const int grid = std::min(f.n_chunks, f.n_cu * 16);
  OutT* o = static_cast<OutT*>(out);
  const uint32_t inside = f.mobius_in ? ~0u : 0u;
  if (f.red_rows == 1)
    hipLaunchKernelGGL((high_reduce_kernel<OutT, 1>), dim3(grid), dim3(NT), 0, st, f.insts, f.chunks,
                       f.n_chunks, inside, Y, o);
  else if (f.red_rows == 4)
    hipLaunchKernelGGL((high_reduce_kernel<OutT, 4>), dim3(grid), dim3(NT), 0, st, f.insts, f.chunks,
                       f.n_chunks, inside, Y, o);
  else
    hipLaunchKernelGGL((high_reduce_kernel<OutT, 16>), dim3(grid), dim3(NT), 0, st, f.insts, f.chunks,
                       f.n_chunks, inside, Y, o);
  return hipGetLastError();
}
hipError_t launch_high_reduce(const HighLaunch& f, const double* Y, void* out, hipStream_t st) {
  return f.prec == PREC_F64 ? launch_high_reduce_t<double>(f, Y, out, st)
                            : launch_high_reduce_t<float>(f, Y, out, st);
}

template <int L, typename SwT, typename MobT, bool IN64>
static hipError_t config_high_l() {
  constexpr int lds = LdsHigh<L, SwT, MobT>::bytes;
  hipError_t e = hipFuncSetAttribute(
      reinterpret_cast<const void*>(tile_high_kernel<L, SwT, MobT, IN64, wpe_high<SwT>(), false>),
      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(
      reinterpret_cast<const void*>(tile_high_kernel<L, SwT, MobT, IN64, wpe_high<SwT>(), true>),
      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}
template <typename SwT, typename MobT, bool IN64>
static hipError_t config_high_t() {
  const hipError_t e = config_high_l<5, SwT, MobT, IN64>();
  return e != hipSuccess ? e : config_high_l<6, SwT, MobT, IN64>();
}
hipError_t configure_high(int prec) {
  switch (prec) {
    case PREC_F32: return config_high_t<float, float, false>();
    case PREC_F32_COMP: return config_high_t<float, TwoFN, false>();
    case PREC_F32_FP64MOB: return config_high_t<float, double, false>();
    case PREC_F64: return config_high_t<double, double, true>();
  }
  return hipErrorInvalidValue;
}

}  // namespace fsi
