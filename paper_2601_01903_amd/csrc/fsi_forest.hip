// Value function of a tree ensemble on the GPU (include/fsi_forest.h):
// v(S) = (1/B) sum_b sum_k f_k(z_b(S)) for all 2^d coalitions S, the input
// the FSI operator consumes (Sec. 2.1 value function; the paper's appendix
// times this step separately in its bottleneck analysis).
//
// Per call, a small kernel folds the explained point and the background
// points into every internal node: the node's decision when its feature is
// in S (x_f >= threshold, one bit) and, for each background b, when it is not
// (bg_b,f >= threshold, one bit per background in a 32-bit word). A walk
// then needs no feature values: at a node with feature f, coalition S goes
// right iff (S >> f & 1) ? dx : (bits >> b & 1).
//
// The walk kernels list, per block of coalitions and (background, tree) pair,
// the few leaves its coalitions can reach, let each coalition pick its leaf
// from that list and sum the leaf outputs in FP64 in ascending order of the
// pairs. Node records are 16 bytes (a 200-tree depth-6 forest is 400 KB, held
// in L2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/fsi_forest.h"
#include "fsi_abi.h"
#include "fsi_butterfly_dev.h"
#include "fsi_internal.h"

namespace fsi {
namespace forest {

constexpr int kThreads = 256;
constexpr int kBgChunk = 32;     // backgrounds per decision word
constexpr int kMaxBg = 4096;
constexpr int kMaxDepth = 64;

// code: feature | (x_f >= threshold) << 8 for an internal node, -1 for a leaf
struct alignas(16) Node {
  int32_t code, left, right;
  uint32_t bits;                 // bit j: background (32 c + j) goes right
};

__global__ void __launch_bounds__(kThreads)
prep_kernel(const int32_t* __restrict__ feature, const double* __restrict__ threshold,
            const int32_t* __restrict__ left, const int32_t* __restrict__ right,
            int n_nodes, int d, const double* __restrict__ x, const double* __restrict__ bg,
            int n_bg, Node* __restrict__ out, int32_t* __restrict__ over) {
  if (over && blockIdx.x == 0 && threadIdx.x == 0) *over = 0;   // counted by reach_kernel
  const int n_chunks = (n_bg + kBgChunk - 1) / kBgChunk;
  const int64_t total = (int64_t)n_chunks * n_nodes;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kThreads) {
    const int c = (int)(i / n_nodes);
    const int node = (int)(i - (int64_t)c * n_nodes);
    const int f = feature[node];
    Node p;
    if (f < 0) {
      p.code = -1; p.left = 0; p.right = 0; p.bits = 0;
    } else {
      const double th = threshold[node];
      const int b0 = c * kBgChunk;
      const int nb = min(kBgChunk, n_bg - b0);
      uint32_t bits = 0;
      for (int j = 0; j < nb; ++j)
        bits |= (uint32_t)(bg[(int64_t)(b0 + j) * d + f] >= th) << j;
      p.code = f | ((x[f] >= th) ? 256 : 0);
      p.left = left[node];
      p.right = right[node];
      p.bits = bits;
    }
    out[i] = p;
  }
}

// ---- walk route ----
// A workgroup owns a block of 2^m consecutive coalitions, which share their
// bits from m up. For one background and one tree most nodes are then
// decided for the whole block: x and the background fall on the same side
// of the threshold, the feature is one of the shared bits, or the path has
// already fixed it. What is left is a short list of reachable leaves, each
// with the low bits a coalition must have and must not have, and a coalition
// takes the one leaf whose bits it matches. With thresholds spread like the
// points, 200 depth-6 trees on 20 features leave 2.5 leaves a tree and block
// of 1024 coalitions, against 6 dependent node loads a coalition for a walk
// of its own.
//
// Per chunk of (background, tree) pairs, one thread per pair lists the
// leaves of its pair into LDS (need bits and FP64 outputs); then the
// coalitions test the lists and add the leaf outputs pair by pair, in the
// order of the pairs, so v is bitwise the sum of the plain walk. A pair with
// more than NK leaves in a block is walked per coalition instead.

// need word of a leaf: bit f for a feature f < m that must be in S, bit
// 16 + f for one that must not be; a coalition matches iff
// (need & ~X(S)) == 0 with X(S) = S_low | ~S_low << 16.

// LDS of a chunk of NP pairs: NK need words, the leaf count and the root per
// pair (row of NK + 2 words, read as 8-byte words), then the leaf outputs in
// rows of NK + 1 (odd, so that the threads of a wave write distinct banks).
template <int NP, int NK>
struct LeafLists {
  static constexpr int kNeedRow = NK + 2;
  static constexpr int kValRow = NK + 1;
  uint2 need2[NP * kNeedRow / 2];
  double val[NP * kValRow];
  __device__ __forceinline__ uint32_t* need() { return reinterpret_cast<uint32_t*>(need2); }
};

// Leaves of one tree reachable inside the block (depth-first over the
// choices at undecided nodes; each leaf is reached by a walk from the root
// that follows the recorded choices). Returns the count, NK + 1 if more.
template <int NK>
__device__ __forceinline__ int list_leaves(const Node* __restrict__ P, const double* __restrict__ value,
                                           int root, int jb, int m, uint32_t shared_bits,
                                           uint32_t* __restrict__ need_row, double* __restrict__ val_row) {
  uint32_t choice = 0;   // bit k: the k-th undecided feature of the path is in S
  int depth = 0, n = 0;
  for (;;) {
    int node = root, k = 0;
    uint32_t need = 0;
    for (;;) {
      const Node w = P[node];
      if (w.code < 0) break;
      const uint32_t dx = ((uint32_t)w.code >> 8) & 1u, db = (w.bits >> jb) & 1u;
      uint32_t go = dx;
      if (dx != db) {
        const uint32_t f = (uint32_t)w.code & 255u;
        uint32_t in;
        if ((int)f >= m) {
          in = (shared_bits >> f) & 1u;
        } else if ((need >> f) & 0x10001u) {
          in = (need >> f) & 1u;
        } else {
          if (k == depth) { choice &= ~(1u << k); ++depth; }
          in = (choice >> k) & 1u;
          need |= in ? 1u << f : 0x10000u << f;
          ++k;
        }
        go = in ? dx : db;
      }
      node = go ? w.right : w.left;
    }
    if (n == NK) return NK + 1;
    need_row[n] = need;
    val_row[n] = value[node];
    ++n;
    while (depth > 0 && ((choice >> (depth - 1)) & 1u)) --depth;
    if (depth == 0) return n;
    choice |= 1u << (depth - 1);
  }
}

// Leaves of a pair reachable by any coalition at all, over the d bits: in must
// be in S, out must not. Entry i of pair g at i * pairs + g, counts in cnt.
// Made once per call, so a block only picks the ones its shared bits allow
// instead of walking the tree again. A pair with more than 64 of them has no
// list, and its coalitions walk. (Listing such a pair's leaves in every block
// instead, by one thread, is a chain of up to 13 walks that the block waits for:
// 20 depth-12 trees at d = 20, x and background apart everywhere: 337 us, 178 by
// plain walks.) The blocks do list those of up to 64 that find no row where the
// pairs are too many for 64 rows each.
constexpr int kReachMax = 64, kReachMin = 24;   // rows, as the workspace allows
constexpr int kListMax = 12;     // leaves of a block's list
struct alignas(16) Reach {
  uint32_t in, out;
  double value;
};
struct ReachLists {
  const Reach* leaf;
  const int32_t* cnt;      // null: no lists (each block makes its own)
  const int32_t* over;     // lists overflow in about over / kSamples pairs of a block
  int rows;
};

// A wave per pair takes the tree level by level from its root: lane i holds
// the i-th node that some coalition reaches on the level, with the bits that it
// takes to get there, and a node whose feature is undecided gives two. Past 64
// of them the wave stops: a pair costs its depth in dependent loads, whatever
// the number of leaves (by root-to-leaf paths, 64 at a time, a call with one
// depth-14 tree at d = 10 took 811 us; now 23).
//
// What the lists of the blocks (m low bits) will hold is counted for kSamples
// settings of their shared bits.
constexpr int kSamples = 4;
__global__ void __launch_bounds__(kThreads)
reach_kernel(const Node* __restrict__ prep, const double* __restrict__ value,
             const int32_t* __restrict__ roots, int n_trees, int n_nodes, int64_t pairs, int m,
             int rows, Reach* __restrict__ leaf, int32_t* __restrict__ cnt, int32_t* __restrict__ over) {
  struct At { int32_t node; uint32_t in, out; };
  __shared__ At next[kThreads / 64][128];
  const int lane = threadIdx.x & 63;
  const uint32_t high = ~0u << m;
  At* N = next[threadIdx.x >> 6];
  int32_t n_over = 0;
  const int64_t wave0 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  for (int64_t g = wave0; g < pairs; g += (int64_t)gridDim.x * (kThreads / 64)) {
    const int b = (int)(g / n_trees), t = (int)(g - (int64_t)b * n_trees);
    const Node* P = prep + (int64_t)(b / kBgChunk) * n_nodes;
    const int jb = b % kBgChunk;
    At at{roots[t], 0u, 0u};
    int n = 1;
    while (n <= 64) {
      bool inner = false, both = false;
      At dn{};                       // the other child, taken without the feature
      if (lane < n) {
        const Node w = P[at.node];
        inner = w.code >= 0;
        if (inner) {
          const uint32_t bit = 1u << ((uint32_t)w.code & 255u);
          const uint32_t dx = ((uint32_t)w.code >> 8) & 1u, db = (w.bits >> jb) & 1u;
          both = dx != db && !((at.in | at.out) & bit);
          dn = At{db ? w.right : w.left, at.in, both ? at.out | bit : at.out};
          if (both) at.in |= bit;
          at.node = ((at.out & bit) ? db : dx) ? w.right : w.left;
        }
      }
      if (!__ballot(inner)) break;   // all leaves
      const uint64_t two = __ballot(both);
      const int k = lane + __popcll(two & ((1ull << lane) - 1ull));
      if (lane < n) {
        N[k] = at;
        if (both) N[k + 1] = dn;
      }
      // the wave reads what its own lanes wrote
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      n += __popcll(two);
      if (lane < n) at = N[lane];
      __builtin_amdgcn_wave_barrier();
    }
    int overs = 0;
    uint32_t s = (uint32_t)g * 0x9e3779b9u;
#pragma unroll
    for (int k = 0; k < kSamples; ++k) {
      s = (s ^ (s >> 15)) * 0x85ebca6bu + 0x6a09e667u;
      const uint32_t S = s ^ (s >> 13);
      const int hit = __popcll(__ballot(lane < n && !(((at.in & ~S) | (at.out & S)) & high)));
      overs += n > 64 || hit > kListMax;     // past 64 the pair is walked
    }
    n_over += overs;
    if (n <= rows && lane < n) leaf[(int64_t)lane * pairs + g] = Reach{at.in, at.out, value[at.node]};
    if (lane == 0) cnt[g] = n;
  }
  if (lane == 0 && n_over) atomicAdd(over, n_over);
}

// One chunk: pairs [g0, g0 + np) of the (background, tree) sequence.
template <int NP, int NK>
__device__ __forceinline__ void build_lists(const Node* __restrict__ prep, const double* __restrict__ value,
                                            const int32_t* __restrict__ roots, int n_trees,
                                            int n_nodes, const ReachLists& reach, int64_t pairs,
                                            int64_t g0, int np, int m, uint32_t shared_bits,
                                            LeafLists<NP, NK>& L) {
  const int p = threadIdx.x;
  if (p >= np) return;
  const int64_t g = g0 + p;
  const int b = (int)(g / n_trees);
  const int root = roots[(int)(g - (int64_t)b * n_trees)];
  uint32_t* row = L.need() + p * LeafLists<NP, NK>::kNeedRow;
  const int all = reach.cnt ? reach.cnt[g] : 0;
  if (0 < all && all <= reach.rows) {
    double* vrow = L.val + p * LeafLists<NP, NK>::kValRow;
    const uint32_t low = (1u << m) - 1u;
    int n = 0;
    for (int i = 0; i < all; i += 4) {
      Reach e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) e[q] = reach.leaf[(int64_t)min(i + q, all - 1) * pairs + g];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (i + q >= all || (e[q].in & ~low & ~shared_bits) || (e[q].out & ~low & shared_bits)) continue;
        if (n < NK) {
          row[n] = (e[q].in & low) | (e[q].out & low) << 16;
          vrow[n] = e[q].value;
        }
        ++n;
      }
    }
    row[NK] = (uint32_t)min(n, NK + 1);
    row[NK + 1] = (uint32_t)root;
    return;
  }
  if (all > kReachMax) {         // walk
    row[NK] = NK + 1;
    row[NK + 1] = (uint32_t)root;
    return;
  }
  row[NK] = (uint32_t)list_leaves<NK>(prep + (int64_t)(b / kBgChunk) * n_nodes, value, root,
                                      b % kBgChunk, m, shared_bits, row,
                                      L.val + p * LeafLists<NP, NK>::kValRow);
  row[NK + 1] = (uint32_t)root;
}

// Plain walks (pairs with more leaves than a list holds): K of them a thread, so
// that their dependent loads overlap; at: the roots, then the leaves. depth: the
// forest's, after which every node is a leaf and need not be read.
template <int K>
__device__ __forceinline__ void walk(const Node* const (&P)[K], const int (&jb)[K], const uint32_t (&S)[K],
                                     int depth, int (&at)[K]) {
  bool inner = true;
  for (int lv = 0; lv < depth && __any(inner); ++lv) {
    Node w[K];
#pragma unroll
    for (int j = 0; j < K; ++j) w[j] = P[j][at[j]];
    inner = false;
#pragma unroll
    for (int j = 0; j < K; ++j)
      if (w[j].code >= 0) {
        const uint32_t f = (uint32_t)w[j].code & 255u;
        const uint32_t go = ((S[j] >> f) & 1u) ? ((uint32_t)w[j].code >> 8) & 1u : (w[j].bits >> jb[j]) & 1u;
        at[j] = go ? w[j].right : w[j].left;
        inner = true;
      }
  }
}

// The lists of 64 pairs, one per lane, as a wave reads them: the first four
// need words and the count.
struct LaneLists {
  uint32_t nd[4], cnt;
};
template <int NP, int NK>
__device__ __forceinline__ LaneLists lane_lists(LeafLists<NP, NK>& L, int p) {
  constexpr int R2 = LeafLists<NP, NK>::kNeedRow / 2;
  const uint2 a = L.need2[p * R2], b = L.need2[p * R2 + 1];
  return LaneLists{{a.x, a.y, b.x, b.y}, L.need2[p * R2 + NK / 2].x};
}
// Index in pair p's list of the leaf each of KP coalitions takes (nx = ~X);
// q: p's lane in ll. The pair and its list are uniform in the wave.
template <int NP, int NK, int KP>
__device__ __forceinline__ void match(LeafLists<NP, NK>& L, const LaneLists& ll, int p, int q, int n,
                                      const uint32_t (&nx)[KP], int (&idx)[KP]) {
#pragma unroll
  for (int j = 0; j < KP; ++j) idx[j] = n - 1;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < n - 1) {
      const uint32_t need = (uint32_t)__builtin_amdgcn_readlane((int)ll.nd[i], q);
#pragma unroll
      for (int j = 0; j < KP; ++j) idx[j] = (need & nx[j]) == 0u ? i : idx[j];
    }
  for (int i = 4; i < n - 1; ++i) {
    const uint32_t need = L.need()[p * LeafLists<NP, NK>::kNeedRow + i];
#pragma unroll
    for (int j = 0; j < KP; ++j) idx[j] = (need & nx[j]) == 0u ? i : idx[j];
  }
}

// Every thread owns KP coalitions, base + tid + j * kThreads. Pairs without a
// list are walked, eight walks a thread at once where they follow each other
// (d = 20, x and background apart everywhere: 20 depth-12 trees 614 us one walk at
// a time and listed first, now 160, plain walks 179; 50 depth-10 trees 585, now
// 309, 342).
template <typename OutT, int KP>
__global__ void __launch_bounds__(kThreads)
walk_wide_kernel(const Node* __restrict__ prep, const double* __restrict__ value,
                 const int32_t* __restrict__ roots, int n_trees, int n_nodes, int depth, ReachLists reach,
                 int n_bg, int d, int m, OutT* __restrict__ v) {
  constexpr int NP = kThreads, NK = kListMax;
  __shared__ LeafLists<NP, NK> L;
  const uint32_t base = (uint32_t)blockIdx.x * (kThreads * KP);
  const int lane = threadIdx.x & 63;
  uint32_t nx[KP];
  double acc[KP];
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    const uint32_t low = (threadIdx.x + j * kThreads) & ((1u << m) - 1u);
    nx[j] = ~low & 0xffffu;
    nx[j] |= low << 16;
    acc[j] = 0.0;
  }
  const int64_t total = (int64_t)n_bg * n_trees;
  for (int64_t g0 = 0; g0 < total; g0 += NP) {
    const int np = (int)min((int64_t)NP, total - g0);
    build_lists<NP, NK>(prep, value, roots, n_trees, n_nodes, reach, total, g0, np, m, base, L);
    __syncthreads();
    for (int p0 = 0; p0 < np; p0 += 64) {
      const LaneLists ll = lane_lists<NP, NK>(L, min(p0 + lane, np - 1));
      const int nq = min(64, np - p0);
      for (int q = 0; q < nq; ++q) {
        const int p = p0 + q;
        const int n = __builtin_amdgcn_readlane((int)ll.cnt, q);
        if (n > NK) {
          // where 8 / KP pairs in a row have no list, eight walks in flight
          auto walk_pairs = [&](auto rc) {
            constexpr int R = decltype(rc)::value;
            const Node* P[R * KP];
            int jb[R * KP], at[R * KP];
            uint32_t S[R * KP];
#pragma unroll
            for (int r = 0; r < R; ++r) {
              const int b = (int)((g0 + p + r) / n_trees);
              const int root = (int)L.need()[(p + r) * LeafLists<NP, NK>::kNeedRow + NK + 1];
#pragma unroll
              for (int j = 0; j < KP; ++j) {
                P[r * KP + j] = prep + (int64_t)(b / kBgChunk) * n_nodes;
                jb[r * KP + j] = b % kBgChunk;
                at[r * KP + j] = root;
                S[r * KP + j] = base | (nx[j] >> 16);
              }
            }
            walk<R * KP>(P, jb, S, depth, at);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
              for (int j = 0; j < KP; ++j) acc[j] += value[at[r * KP + j]];
          };
          constexpr int R = 8 / KP;
          const uint64_t run = __ballot(lane < nq && ll.cnt > (uint32_t)NK) >> q;
          if (R > 1 && (run & ((1u << R) - 1u)) == (1u << R) - 1u) {
            walk_pairs(std::integral_constant<int, R>{});
            q += R - 1;
          } else {
            walk_pairs(std::integral_constant<int, 1>{});
          }
        } else {
          const double* row = L.val + p * LeafLists<NP, NK>::kValRow;
          if (n == 1) {   // the whole block takes one leaf
            const double x = row[0];
#pragma unroll
            for (int j = 0; j < KP; ++j) acc[j] += x;
            continue;
          }
          int idx[KP];
          match<NP, NK, KP>(L, ll, p, q, n, nx, idx);
#pragma unroll
          for (int j = 0; j < KP; ++j) acc[j] += row[idx[j]];
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    const uint32_t s = base + threadIdx.x + j * kThreads;
    if (s < (1u << d)) v[s] = (OutT)(acc[j] / (double)n_bg);
  }
}

// Few coalitions: a workgroup owns 64 of them and runs the pairs as a
// pipeline over three buffers of lists: in one step four waves list a chunk,
// six match the chunk before (leaving each coalition's leaf in LDS, one byte
// per pair: its offset in the list) and one adds the outputs of the chunk
// before that, in the order of the pairs. The sums are one chain per coalition
// (5000 additions at 50 trees and 100 backgrounds) and a wave issues an
// instruction every four to five clocks, so that wave shares its SIMD with a
// listing wave only (the roles go by wave number, SIMD = wave % 4), and the
// matching waves the other three. 50 trees, d = 14, 100 backgrounds: 185 us
// with the three parts in turns, 142 with a matching wave beside the adding
// one, now 114. Where many pairs have no list, the waves walk instead (see
// kWalkShare; 50 depth-12 trees, two backgrounds, d = 16, x and background apart
// everywhere: 1240 us by the adding wave, 433 by a kernel of plain walks, now 102).
constexpr int kNarrowPairs = 256;
constexpr int kNarrowThreads = 768;
constexpr int kAddWave = 4;        // waves 0-3 list, 8 idles, the other six match
// A pair without a list is walked by the adding wave alone, 4 us each; past one in
// kWalkShare of them every wave walks, listed pairs too (1000 depth-3 trees and n
// of depth 9 that overflow, two backgrounds, d = 14: 92 us at n = 5, 222 at 20;
// with every wave walking 167 at 30, 312 without that).
constexpr int kWalkShare = 50;
template <typename OutT>
__global__ void __launch_bounds__(kNarrowThreads)
walk_narrow_kernel(const Node* __restrict__ prep, const double* __restrict__ value,
                   const int32_t* __restrict__ roots, int n_trees, int n_nodes, int depth, ReachLists reach,
                   int n_bg, int d, OutT* __restrict__ v) {
  constexpr int NP = kNarrowPairs, NK = kListMax;
  constexpr int VR = LeafLists<NP, NK>::kValRow;
  __shared__ LeafLists<NP, NK> lists[3];
  // byte i: 8 x leaf index of pair 16 r + i (255: walk)
  __shared__ uint4 picks[2][NP / 16][64];
  __shared__ uint32_t unlisted[2][NP / 16];   // pairs 16 r .. 16 r + 15 hold one without a list
  const int m = min(d, 6);
  const uint32_t base = (uint32_t)blockIdx.x << 6;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t low = (uint32_t)lane & ((1u << m) - 1u);
  const uint32_t nx[1] = {(~low & 0xffffu) | (low << 16)};
  double acc = 0.0;
  const int64_t total = (int64_t)n_bg * n_trees;
  const bool walks = reach.over && (int64_t)*reach.over * kWalkShare > total * kSamples;
  const int64_t chunks = walks ? 0 : (total + NP - 1) / NP;
  if (walks) {
    // every wave but the adding one walks 8 pairs at a time into LDS, while
    // that one adds the pairs before
    constexpr int W = kNarrowThreads / 64 - 1, PP = 8 * W;
    static_assert(sizeof(double) * 2 * PP * 64 <= sizeof(lists), "leaf outputs over the lists");
    double* out2 = reinterpret_cast<double*>(lists);
    const int64_t steps = (total + PP - 1) / PP;
    for (int64_t it = 0; it <= steps; ++it) {
      const int64_t g0 = it * PP + 8 * (wave - (wave > kAddWave));
      if (wave == kAddWave) {
        const int np = (int)min((int64_t)PP, total - (it - 1) * PP);
        const double* x = out2 + ((it - 1) & 1) * PP * 64 + lane;
        if (it > 0) {
#pragma unroll 8
          for (int p = 0; p < np; ++p) acc += x[p * 64];
        }
      } else if (g0 < total) {
        const Node* P[8];
        int jb[8], at[8];
        uint32_t S[8];
        int b = (int)(g0 / n_trees), t = (int)(g0 - (int64_t)b * n_trees);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          P[q] = prep + (int64_t)(b / kBgChunk) * n_nodes;
          jb[q] = b % kBgChunk;
          at[q] = roots[t];
          S[q] = base | low;
          if (g0 + q + 1 < total && ++t == n_trees) { t = 0; ++b; }   // past the end: the last pair again
        }
        walk<8>(P, jb, S, depth, at);
        double* x = out2 + (it & 1) * PP * 64 + (int)(g0 - it * PP) * 64 + lane;
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q * 64] = value[at[q]];
      }
      __syncthreads();
    }
  }
  for (int64_t it = 0; it < chunks + 2 && !walks; ++it) {
    if (wave < NP / 64) {
      const int64_t g0 = it * NP;
      if (it < chunks)
        build_lists<NP, NK>(prep, value, roots, n_trees, n_nodes, reach, total, g0,
                            (int)min((int64_t)NP, total - g0), m, base, lists[it % 3]);
    } else if (wave % 4 != 0) {
      // groups of 16 pairs, dealt to the six waves
      const int64_t c = it - 1;
      const int np = c >= 0 && c < chunks ? (int)min((int64_t)NP, total - c * NP) : 0;
      LeafLists<NP, NK>& L = lists[(c + 3) % 3];
      for (int p0 = 16 * (wave % 4 - 1 + 3 * (wave / 8)); p0 < np; p0 += 16 * 6) {
        const LaneLists ll = lane_lists<NP, NK>(L, min(p0 + (lane & 15), np - 1));
        const int nq = min(16, np - p0);
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int q = min(i, nq - 1);
          const int n = __builtin_amdgcn_readlane((int)ll.cnt, q);
          if (n > NK) {
            w[i >> 2] |= 255u << (8 * (i & 3));
          } else if (n > 1) {
            int idx[1];
            match<NP, NK, 1>(L, ll, p0 + q, q, n, nx, idx);
            w[i >> 2] |= (uint32_t)idx[0] << (8 * (i & 3) + 3);
          }
        }
        picks[c & 1][p0 >> 4][lane] = uint4{w[0], w[1], w[2], w[3]};
        const uint64_t over = __ballot(lane < nq && ll.cnt > (uint32_t)NK);
        if (lane == 0) unlisted[c & 1][p0 >> 4] = over != 0;
      }
    } else if (wave == kAddWave && it >= 2) {
      const int64_t c = it - 2, g0 = c * NP;
      const int np = (int)min((int64_t)NP, total - g0);
      LeafLists<NP, NK>& L = lists[c % 3];
      const uint4 (*pick)[64] = picks[c & 1];
      // every LDS read of 16 pairs in flight while the 16 before are added
      // (read by read, one pair waited for the one before: 400 us)
      const int full = np / 16;              // whole groups of 16 pairs
      const uint32_t bad = (uint32_t)__ballot(lane < full && unlisted[c & 1][lane & (NP / 16 - 1)]);
      double x[2][16];
      auto fetch = [&](int g, double (&y)[16]) {
        const uint4 u = pick[g][lane];
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
        const unsigned char* row = reinterpret_cast<const unsigned char*>(L.val + g * 16 * VR);
#pragma unroll
        for (int i = 0; i < 16; ++i)
          y[i] = *reinterpret_cast<const double*>(row + ((w[i >> 2] >> (8 * (i & 3))) & 255u) + i * VR * 8);
      };
      // the groups in runs that have a list for every pair, and pair by pair
      // those that have not
      for (int g = 0; g * 16 < np;) {
        const int end = g >= full ? g : min(full, g + __builtin_ctz((bad >> g) | 0x10000u));
        if (g < end) fetch(g, x[0]);
        for (; g < end; g += 2) {
          if (g + 1 < end) fetch(g + 1, x[1]);
#pragma unroll
          for (int i = 0; i < 16; ++i) acc += x[0][i];
          if (g + 1 >= end) break;
          if (g + 2 < end) fetch(g + 2, x[0]);
#pragma unroll
          for (int i = 0; i < 16; ++i) acc += x[1][i];
        }
        g = end;
        for (int p = g * 16; p < min(np, g * 16 + 16); ++p) {
          const uint4 u = pick[p >> 4][lane];
          const uint32_t w = (p & 8) ? ((p & 4) ? u.w : u.z) : ((p & 4) ? u.y : u.x);
          const uint32_t o = (w >> (8 * (p & 3))) & 255u;
          if (o != 255u) {
            acc += L.val[p * VR + (o >> 3)];
          } else {   // the pair has no list (uniform)
            const int b = (int)((g0 + p) / n_trees);
            const Node* P[1] = {prep + (int64_t)(b / kBgChunk) * n_nodes};
            const int jb[1] = {b % kBgChunk};
            const uint32_t S[1] = {base | low};
            int at[1] = {(int)L.need()[p * LeafLists<NP, NK>::kNeedRow + NK + 1]};
            walk<1>(P, jb, S, depth, at);
            acc += value[at[0]];
          }
        }
        ++g;
      }
    }
    __syncthreads();
  }
  if (wave == kAddWave) {
    const uint32_t s = base + (uint32_t)lane;
    if (s < (1u << d)) v[s] = (OutT)(acc / (double)n_bg);
  }
}

// A few short walks: two coalitions a thread, no lists (whose pass is a launch
// of its own).
constexpr int kPlainKP = 2;
template <typename OutT>
__global__ void __launch_bounds__(kThreads)
walk_plain_kernel(const Node* __restrict__ prep, const double* __restrict__ value,
                  const int32_t* __restrict__ roots, int n_trees, int n_nodes, int depth, int n_bg,
                  int d, OutT* __restrict__ v) {
  constexpr int KP = kPlainKP;
  const uint32_t s0 = blockIdx.x * (kThreads * KP) + threadIdx.x;
  uint32_t S[KP];
  double acc[KP];
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    S[j] = (s0 + j * kThreads) & ((1u << d) - 1u);   // past the end: a valid one, not stored
    acc[j] = 0.0;
  }
  for (int b = 0; b < n_bg; ++b)
    for (int t = 0; t < n_trees; ++t) {
      const Node* P[KP];
      int jb[KP], at[KP];
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        P[j] = prep + (int64_t)(b / kBgChunk) * n_nodes;
        jb[j] = b % kBgChunk;
        at[j] = roots[t];
      }
      walk<KP>(P, jb, S, depth, at);
#pragma unroll
      for (int j = 0; j < KP; ++j) acc[j] += value[at[j]];
    }
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    const uint32_t s = s0 + j * kThreads;
    if (s < (1u << d)) v[s] = (OutT)(acc[j] / (double)n_bg);
  }
}

// Plain walks for up to four pairs or 32 dependent loads in all, and for fewer
// where the walks fill the machine (plain / with lists, in us: 8 depth-3 trees d = 3
// to 18 11 to 13 / 13, 16 of them 18 to 24 / 13; 4 depth-6 trees 11 to 14 / 14; 4 of
// depth 10 with x and background apart everywhere, d = 16, 21 / 25, uniform points
// 21 / 15; d = 20: 8 depth-3 trees 22 / 13, 2 depth-6 trees 13 / 14 to 24).
bool walk_plain(int d, int64_t pairs, int depth) {
  const int64_t loads = pairs * std::max(depth, 1);
  return d < 20 ? pairs <= 4 || loads <= 32 : loads <= 12 >> std::min(d - 20, 4);
}

// Coalitions per thread of the wide kernel, 0 for the narrow one: the most, up to
// eight, that still give every CU four workgroups, what its LDS holds (100 depth-6
// trees d = 21 70 us with eight, 82 with four; 200 d = 20 101 with eight, 90 with
// four; 200 d = 19 73 with four, 69 with two, with no list that suffices 211 and 150;
// d = 18 58 with two, 57 with one, 156 and 106). The narrow kernel takes one workgroup
// per CU and 64 coalitions, up to four rounds of them (50 depth-4 trees, 100
// backgrounds: d = 16 wide 818 us, narrow 445; d = 17 wide 831, narrow 844). Its
// pipeline fills and drains in each round, so at two and four rounds (d = 15, 16)
// it takes some pairs to be worth it (depth 6, d = 16: 16 trees narrow 29 us, wide 14,
// 128 trees 43 and 34, where no list suffices 88 and 79; 64 such trees of depth
// 10: 56 and 85. d = 15: 16 trees 20 and 14, 64 trees 23 and 24).
int walk_kp(int d, int64_t pairs) {
  if (d >= 18) return 1 << std::min(d - 18, 3);
  return d >= 17 || (d >= 15 && pairs <= (d == 15 ? 16 : 64)) ? 1 : 0;
}

// bits of a block's coalitions
int walk_bits(int d, int kp) {
  return kp == 0 ? std::min(d, 6) : kp == 8 ? 11 : kp == 4 ? 10 : kp == 2 ? 9 : 8;
}

template <typename OutT>
void launch_walk(const Node* prep, const double* value, const int32_t* roots, int n_trees,
                 int n_nodes, int depth, const ReachLists& reach, bool plain, int kp, int n_bg, int d,
                 OutT* v, hipStream_t st) {
  if (plain) {
    const int grid = ((1 << d) + kThreads * kPlainKP - 1) / (kThreads * kPlainKP);
    walk_plain_kernel<OutT><<<grid, kThreads, 0, st>>>(prep, value, roots, n_trees, n_nodes, depth, n_bg,
                                                       d, v);
    return;
  }
  if (kp == 0) {
    const int grid = d > 6 ? 1 << (d - 6) : 1;
    walk_narrow_kernel<OutT><<<grid, kNarrowThreads, 0, st>>>(prep, value, roots, n_trees, n_nodes, depth,
                                                              reach, n_bg, d, v);
    return;
  }
  const int m = walk_bits(d, kp);
  auto* kernel = kp == 1 ? walk_wide_kernel<OutT, 1> : kp == 2 ? walk_wide_kernel<OutT, 2>
               : kp == 4 ? walk_wide_kernel<OutT, 4> : walk_wide_kernel<OutT, 8>;
  kernel<<<1 << (d - m), kThreads, 0, st>>>(prep, value, roots, n_trees, n_nodes, depth, reach, n_bg, d, m,
                                            v);
}

// ---- Moebius route ----
// A leaf of a tree is reached at z_b(S) iff every test on its root path
// passes. With alpha_f (beta_f) = [x (bg_b) passes every test on feature f of
// the path], the leaf's indicator is prod_f (beta_f + [f in S](alpha_f -
// beta_f)), whose Moebius coefficients sit on R = I u Q: I = {f: beta_f = 0}
// (unreachable if some f in I has alpha_f = 0), Q any subset of
// Fr = {f: beta_f = 1, alpha_f = 0}, with sign (-1)^|Q|; value / B * (-1)^|Q|
// is added at every such R.
// Zeroes 2^d entries, 16 bytes a store (d = 0 does not occur).
__global__ void __launch_bounds__(kThreads)
fill_kernel(double2* __restrict__ a, int64_t n2) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n2;
       i += (int64_t)gridDim.x * kThreads)
    a[i] = double2{0.0, 0.0};
}

// One thread per path and group of kScatterBg backgrounds: the path's nodes
// and thresholds are read once per group, the points' coordinates from LDS.
// Most coefficients fall on a few small sets (every tree and background adds
// one at the empty set), and FP64 atomics on one address serialise in
// memory: a workgroup collects the sets of at most two players in LDS (index
// 0, then 1 + i, then 1 + d + C(j, 2) + i for i < j) and adds each to memory
// once at the end. Few (path, background) pairs are reachable at all, and they
// have 1 to 2^|Fr| terms: the workgroup lists the reachable ones in LDS and
// then gives kTermLanes lanes to each (looped over by the thread that found
// them, the terms took 35 of 60 us at 200 depth-6 trees, d = 20, 100
// backgrounds; now the kernel takes 45, half of it the atomics).
constexpr int kScatterBg = 8;
constexpr int kScatterGrid = 256;   // workgroups that collect and flush
constexpr int kScatterFew = 32;     // work items below which the groups shrink
constexpr int kSmallSets = 1 + kMaxD + kMaxD * (kMaxD - 1) / 2;
constexpr int kTermLanes = 4;   // the subsets of two members, see the loop
struct PathTerms {       // a reachable path of one background
  uint32_t I, Fr;
  double c;
};

__global__ void __launch_bounds__(kThreads)
mobius_scatter_kernel(const int32_t* __restrict__ path_off, const int32_t* __restrict__ steps,
                      const int32_t* __restrict__ path_leaf, int n_paths,
                      const int32_t* __restrict__ feature, const double* __restrict__ threshold,
                      const double* __restrict__ value, int d, const double* __restrict__ x,
                      const double* __restrict__ bg, int n_bg, int per, double* __restrict__ a) {
  __shared__ double small[kSmallSets];
  __shared__ double xs[kMaxD], zs[kScatterBg][kMaxD];
  __shared__ PathTerms list[kThreads * kScatterBg];
  __shared__ int n_list;
  const int lane = threadIdx.x & 63;
  const int n_small = 1 + d + d * (d - 1) / 2;
  for (int i = threadIdx.x; i < n_small; i += kThreads) small[i] = 0.0;
  if ((int)threadIdx.x < d) xs[threadIdx.x] = x[threadIdx.x];
  const int chunks = (n_paths + kThreads - 1) / kThreads;    // of paths, per group
  const int groups = (n_bg + per - 1) / per;
  const int64_t total = (int64_t)chunks * groups;
  int g_prev = -1;
  for (int64_t it = blockIdx.x; it < total; it += gridDim.x) {
    const int g = (int)(it / chunks);
    const int p = (int)(it - (int64_t)g * chunks) * kThreads + (int)threadIdx.x;
    const int b0 = g * per;
    const int nb = min(per, n_bg - b0);
    __syncthreads();             // the previous list is used up
    if (threadIdx.x == 0) n_list = 0;
    if (g != g_prev) {           // uniform in the workgroup
      for (int i = threadIdx.x; i < kScatterBg * d; i += kThreads) {
        const int b = i / d;
        zs[b][i - b * d] = bg[(int64_t)(b0 + min(b, nb - 1)) * d + (i - b * d)];
      }
      g_prev = g;
    }
    __syncthreads();
    uint32_t seen = 0, aok = ~0u, bok[kScatterBg];
#pragma unroll
    for (int b = 0; b < kScatterBg; ++b) bok[b] = ~0u;
    const bool on = p < n_paths;
    const int s0 = on ? path_off[p] : 0, s1 = on ? path_off[p + 1] : 0;
    for (int s = s0; s < s1; ++s) {
      const int e = steps[s];
      const int node = e >> 1;
      const bool dir = e & 1;
      const int f = feature[node];
      const double th = threshold[node];
      const uint32_t bit = 1u << f;
      seen |= bit;
      if ((xs[f] >= th) != dir) aok &= ~bit;
#pragma unroll
      for (int b = 0; b < kScatterBg; ++b)
        if ((zs[b][f] >= th) != dir) bok[b] &= ~bit;
    }
    const double c = on ? value[path_leaf[p]] / (double)n_bg : 0.0;
#pragma unroll
    for (int b = 0; b < kScatterBg; ++b) {
      const uint32_t I = seen & ~bok[b];
      const bool ok = on && b < nb && !(I & ~aok);    // reachable
      const uint64_t m = __ballot(ok);
      int base = 0;
      if (lane == 0 && m) base = atomicAdd(&n_list, __popcll(m));
      base = __builtin_amdgcn_readfirstlane(base);
      if (ok)
        list[base + __popcll(m & ((1ull << lane) - 1ull))] =
            PathTerms{I, seen & bok[b] & ~aok, c};
    }
    __syncthreads();
    const int n = n_list;
    for (int i = threadIdx.x / kTermLanes; i < n; i += kThreads / kTermLanes) {
      const PathTerms t = list[i];
      // lane j takes the subsets with bits j of the two lowest members of Fr
      const uint32_t f0 = t.Fr & (0u - t.Fr), f01 = t.Fr & (t.Fr - 1u), f1 = f01 & (0u - f01);
      const uint32_t rest = f01 ^ f1;
      const uint32_t j = threadIdx.x % kTermLanes;
      const uint32_t Q0 = ((j & 1u) ? f0 : 0u) | ((j & 2u) ? f1 : 0u);
      if (((j & 1u) && !f0) || ((j & 2u) && !f1)) continue;
      uint32_t H = 0;
      do {
        const uint32_t Q = Q0 | H, R = t.I | Q;
        const double v = (__popc(Q) & 1) ? -t.c : t.c;
        if (__popc(R) <= 2) {
          int k = 0;
          if (R) {
            const int hi = 31 - __clz((int)R), lo = __ffs((int)R) - 1;
            k = lo == hi ? 1 + lo : 1 + d + hi * (hi - 1) / 2 + lo;
          }
          atomicAdd(small + k, v);
        } else {
          atomicAdd(a + R, v);
        }
        H = (H - rest) & rest;
      } while (H != 0);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < n_small; k += kThreads) {
    if (small[k] == 0.0) continue;
    uint32_t R = 0;
    if (k > d) {
      int j = 1, o = k - 1 - d;
      while (o >= j) o -= j++;
      R = (1u << j) | (1u << o);
    } else if (k > 0) {
      R = 1u << (k - 1);
    }
    atomicAdd(a + R, small[k]);
  }
}

// Backgrounds per group: fewer, down to one, where that makes up to kScatterFew
// work items (10 depth-5 trees, 8 backgrounds, d = 16, x and background apart
// everywhere: two items 38 us, 16 items 18; lines at 16, 128 and 256 items were no
// better over 212 forests). More items flush the small sets more often.
int scatter_bg(int n_bg, int chunks) {
  int per = kScatterBg;
  while (per > 1 && (int64_t)chunks * ((n_bg + per - 1) / per) < kScatterFew) per /= 2;
  return per;
}

// Subset sums (zeta transform, the inverse of the Moebius butterfly): a pass
// over the low 12 bits, then one over at most 8 more bits each; the last pass
// may write the result in the output dtype instead of in place.
struct ZetaAdd {
  __device__ static double op(double hi, double lo) { return hi + lo; }
};

template <typename OutT>
__global__ void __launch_bounds__(kMobThreads)
zeta_low_kernel(const double* a, int d, OutT* out) {          // out may equal a
  __shared__ double m[kMobLds];
  const int nv = 1 << min(d, kMobTileBits);                   // valid elements
  const int64_t base = (int64_t)blockIdx.x << kMobTileBits;
  const int t = mob_field(threadIdx.x, 8);
  double x[kMobElems];
#pragma unroll
  for (int k = 0; k < kMobElems; ++k) {
    const int e = t | (k << 8);
    x[k] = e < nv ? a[base + e] : 0.0;
  }
  mob_exchange<double>(m, x, 8, 0);
  mob_levels<ZetaAdd>(x, 0);
  mob_exchange<double>(m, x, 0, 4);
  mob_levels<ZetaAdd>(x, 0);
  mob_exchange<double>(m, x, 4, 8);
  mob_levels<ZetaAdd>(x, 0);
#pragma unroll
  for (int k = 0; k < kMobElems; ++k) {
    const int e = t | (k << 8);
    if (e < nv) out[base + e] = (OutT)x[k];
  }
}

template <typename OutT>
__global__ void __launch_bounds__(kMobThreads)
zeta_high_kernel(const double* a, int lo, int G, OutT* out) {  // out may equal a
  __shared__ double m[kMobLds];
  const int cb = kMobTileBits - G;
  const int64_t block = blockIdx.x;
  const int64_t base = ((block >> (lo - cb)) << (lo + G)) +
                       ((block & (((int64_t)1 << (lo - cb)) - 1)) << cb);
  const int p0 = min(cb, 8);
  const int t0 = mob_field(threadIdx.x, p0), t1 = mob_field(threadIdx.x, 8);
  double x[kMobElems];
#pragma unroll
  for (int k = 0; k < kMobElems; ++k) x[k] = a[base + mob_high_at(t0 | (k << p0), cb, lo)];
  mob_levels<ZetaAdd>(x, cb - p0);
  if (G > 4) {
    mob_exchange<double>(m, x, p0, 8);
    mob_levels<ZetaAdd>(x, cb - 4);
  }
#pragma unroll
  for (int k = 0; k < kMobElems; ++k)
    out[base + mob_high_at(t1 | (k << 8), cb, lo)] = (OutT)x[k];
}

// The subset sums of a (2^d), the last pass into out.
template <typename OutT>
void launch_zeta(double* a, int d, OutT* out, hipStream_t st) {
  const int high = std::max(0, d - kMobTileBits);
  const int grid = 1 << high;
  if (high == 0) {
    zeta_low_kernel<OutT><<<grid, kMobThreads, 0, st>>>(a, d, out);
    return;
  }
  zeta_low_kernel<double><<<grid, kMobThreads, 0, st>>>(a, d, a);
  const int np = (high + kMobGroup - 1) / kMobGroup;
  for (int p = 0, lo = kMobTileBits; p < np; ++p) {
    const int G = (d - lo + np - p - 1) / (np - p);
    if (p + 1 < np) zeta_high_kernel<double><<<grid, kMobThreads, 0, st>>>(a, lo, G, a);
    else zeta_high_kernel<OutT><<<grid, kMobThreads, 0, st>>>(a, lo, G, out);
    lo += G;
  }
}

// Lists of reachable leaves are kept for forests that need at most this much
// for them.
constexpr size_t kReachBytes = (size_t)64 << 20;

constexpr int kMaxFreeSplits = 24;  // longest path the Moebius route expands
constexpr int64_t kMaxPathSteps = (int64_t)1 << 26;

}  // namespace forest
}  // namespace fsi

using namespace fsi;
using namespace fsi::forest;

struct fsi_forest_s {
  int d = 0, n_trees = 0, n_nodes = 0, max_bg = 0, depth = 0, device = 0;
  unsigned char* arena = nullptr;  // holds the arrays up to path_leaf
  int32_t* feature = nullptr;
  int32_t* left = nullptr;
  int32_t* right = nullptr;
  int32_t* roots = nullptr;
  double* threshold = nullptr;
  double* value = nullptr;
  Node* prep = nullptr;
  // root-to-leaf paths for the Moebius route (n_paths < 0: not available)
  int n_paths = 0, max_path = 0;
  int32_t* path_off = nullptr;
  int32_t* steps = nullptr;        // node << 1 | went right
  int32_t* path_leaf = nullptr;
  Reach* reach = nullptr;          // leaf lists of a walk call (null: not kept)
  int reach_rows = 0;
  int32_t* reach_cnt = nullptr;    // past the lists: pairs, then the overflow count
};

namespace {

fsi_status ffail(fsi_status st, const std::string& msg) {
  record_error(msg);
  return st;
}

void free_forest(fsi_forest_s* F) {
  if (!F) return;
  if (F->arena) (void)hipFree(F->arena);
  if (F->reach) (void)hipFree(F->reach);
  delete F;
}

// Longest root-to-leaf path of the forest in internal nodes, or -1 on a cycle
// or a path longer than kMaxDepth (iterative depth-first search, memoised per
// node; a node is marked while its subtree is open, so meeting a marked node
// means a cycle).
int forest_depth(int n_nodes, const int32_t* feature, const int32_t* left,
                 const int32_t* right, const int32_t* roots, int n_trees) {
  std::vector<int> depth(n_nodes, -2);   // -2 unvisited, -3 on the stack
  int best = 0;
  std::vector<std::pair<int, int>> stack;  // (node, state)
  for (int k = 0; k < n_trees; ++k) {
    stack.push_back({roots[k], 0});
    while (!stack.empty()) {
      auto& [node, state] = stack.back();
      if (feature[node] < 0) { depth[node] = 0; stack.pop_back(); continue; }
      if (state == 0) {
        if (depth[node] >= 0) { stack.pop_back(); continue; }
        if (depth[node] == -3) return -1;          // cycle
        depth[node] = -3;
        state = 1;
        const int l = left[node], r = right[node];
        if (depth[l] == -3 || depth[r] == -3) return -1;
        if (depth[l] == -2) stack.push_back({l, 0});
        if (depth[r] == -2) stack.push_back({r, 0});
        continue;
      }
      const int dl = depth[left[node]], dr = depth[right[node]];
      if (dl < 0 || dr < 0) return -1;
      depth[node] = 1 + std::max(dl, dr);
      if (depth[node] > kMaxDepth) return -1;
      stack.pop_back();
    }
    best = std::max(best, depth[roots[k]]);
  }
  return best;
}

// Every root-to-leaf path (a leaf reached from several roots or along several
// routes counts once per path). Returns false if the paths exceed the caps.
bool enumerate_paths(const int32_t* feature, const int32_t* left, const int32_t* right,
                     const int32_t* roots, int n_trees, std::vector<int32_t>* off,
                     std::vector<int32_t>* steps, std::vector<int32_t>* leaf) {
  off->assign(1, 0);
  steps->clear();
  leaf->clear();
  std::vector<int32_t> path;
  // explicit DFS: (node, next child to visit: 0 left, 1 right, 2 done)
  std::vector<std::pair<int, int>> st;
  for (int k = 0; k < n_trees; ++k) {
    st.assign(1, {roots[k], 0});
    path.clear();
    while (!st.empty()) {
      auto& top = st.back();
      const int node = top.first;
      if (feature[node] < 0) {
        steps->insert(steps->end(), path.begin(), path.end());
        off->push_back((int32_t)steps->size());
        leaf->push_back(node);
        if ((int64_t)steps->size() > kMaxPathSteps || (int64_t)leaf->size() >= ((int64_t)1 << 26))
          return false;
        st.pop_back();
        if (!path.empty()) path.pop_back();
        continue;
      }
      if (top.second == 2) {
        st.pop_back();
        if (!path.empty()) path.pop_back();
        continue;
      }
      const int dir = top.second++;
      path.push_back((node << 1) | dir);
      st.push_back({dir ? right[node] : left[node], 0});
    }
  }
  return true;
}

// Appends an aligned block to a host staging buffer and returns its offset.
template <typename T>
size_t stage(std::vector<unsigned char>& buf, const T* data, size_t n) {
  const size_t off = (buf.size() + 255) & ~(size_t)255;
  buf.resize(off + n * sizeof(T));
  if (n) std::memcpy(buf.data() + off, data, n * sizeof(T));
  return off;
}

}  // namespace

extern "C" {

fsi_status fsi_forest_create(int d, int n_trees, const int32_t* roots, int n_nodes,
                             const int32_t* feature, const double* threshold,
                             const int32_t* left, const int32_t* right, const double* value,
                             int max_bg, fsi_forest_t* out) {
  FSI_ABI_TRY
  if (!out) return ffail(FSI_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (!(1 <= d && d <= kMaxD)) return ffail(FSI_ERR_INVALID_ARG, "need 1 <= d <= 30");
  if (n_trees < 1 || n_nodes < 1) return ffail(FSI_ERR_INVALID_ARG, "need n_trees >= 1 and n_nodes >= 1");
  if (max_bg < 1 || max_bg > kMaxBg) return ffail(FSI_ERR_INVALID_ARG, "need 1 <= max_bg <= 4096");
  if (!roots || !feature || !threshold || !left || !right || !value)
    return ffail(FSI_ERR_INVALID_ARG, "null forest array");
  for (int k = 0; k < n_trees; ++k)
    if (roots[k] < 0 || roots[k] >= n_nodes)
      return ffail(FSI_ERR_INVALID_ARG, "root " + std::to_string(k) + " out of range");
  for (int i = 0; i < n_nodes; ++i) {
    if (feature[i] >= d)
      return ffail(FSI_ERR_INVALID_ARG, "node " + std::to_string(i) + ": feature >= d");
    if (feature[i] >= 0) {
      if (left[i] < 0 || left[i] >= n_nodes || right[i] < 0 || right[i] >= n_nodes)
        return ffail(FSI_ERR_INVALID_ARG, "node " + std::to_string(i) + ": child out of range");
      if (!std::isfinite(threshold[i]))
        return ffail(FSI_ERR_INVALID_ARG, "node " + std::to_string(i) + ": threshold not finite");
    }
  }
  const int depth = forest_depth(n_nodes, feature, left, right, roots, n_trees);
  if (depth < 0)
    return ffail(FSI_ERR_INVALID_ARG, "forest has a cycle or a path of more than 64 splits");
  int dev = 0, n_cu = 0;
  std::string why;
  if (!gfx950_device(&dev, &n_cu, &why)) return ffail(FSI_ERR_UNSUPPORTED, why);

  auto* F = new (std::nothrow) fsi_forest_s();
  if (!F) return ffail(FSI_ERR_OUT_OF_MEMORY, "host allocation failed");
  // frees the partly built forest on every failure below, thrown or returned
  struct Guard {
    fsi_forest_s* f;
    ~Guard() { free_forest(f); }
  } guard{F};
  F->d = d; F->n_trees = n_trees; F->n_nodes = n_nodes; F->max_bg = max_bg; F->depth = depth;
  F->device = dev;
  // leaves keep feature -1 on the device whatever negative value they had
  std::vector<int32_t> feat(feature, feature + n_nodes);
  for (auto& f : feat) f = f < 0 ? -1 : f;
  std::vector<int32_t> poff, psteps, pleaf;
  if (enumerate_paths(feat.data(), left, right, roots, n_trees, &poff, &psteps, &pleaf)) {
    F->n_paths = (int)pleaf.size();
    for (size_t p = 0; p + 1 < poff.size(); ++p)
      F->max_path = std::max(F->max_path, poff[p + 1] - poff[p]);
    if (std::min(F->max_path, d) > kMaxFreeSplits) F->n_paths = -1;
  } else {
    F->n_paths = -1;
  }
  if (F->n_paths < 0) { poff.clear(); psteps.clear(); pleaf.clear(); }
  // one allocation and one copy (ten and nine of them took 100 us more)
  std::vector<unsigned char> buf;
  buf.reserve((size_t)n_nodes * 28 + (poff.size() + psteps.size() + pleaf.size() + n_trees) * 4 + 10 * 256);
  const size_t o_feature = stage(buf, feat.data(), feat.size());
  const size_t o_left = stage(buf, left, (size_t)n_nodes), o_right = stage(buf, right, (size_t)n_nodes);
  const size_t o_roots = stage(buf, roots, (size_t)n_trees);
  const size_t o_threshold = stage(buf, threshold, (size_t)n_nodes);
  const size_t o_value = stage(buf, value, (size_t)n_nodes);
  const size_t o_off = stage(buf, poff.data(), poff.size());
  const size_t o_steps = stage(buf, psteps.data(), psteps.size());
  const size_t o_leaf = stage(buf, pleaf.data(), pleaf.size());
  const size_t chunks = (size_t)((max_bg + kBgChunk - 1) / kBgChunk);
  const size_t o_prep = (buf.size() + 255) & ~(size_t)255;
  hipError_t e = hipMalloc((void**)&F->arena, o_prep + chunks * (size_t)n_nodes * sizeof(Node));
  if (e == hipSuccess) e = hipMemcpy(F->arena, buf.data(), buf.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    auto ints = [&](size_t off) { return reinterpret_cast<int32_t*>(F->arena + off); };
    F->feature = ints(o_feature);
    F->left = ints(o_left);
    F->right = ints(o_right);
    F->roots = ints(o_roots);
    F->threshold = reinterpret_cast<double*>(F->arena + o_threshold);
    F->value = reinterpret_cast<double*>(F->arena + o_value);
    F->path_off = ints(o_off);
    F->steps = ints(o_steps);
    F->path_leaf = ints(o_leaf);
    F->prep = reinterpret_cast<Node*>(F->arena + o_prep);
    // the walk runs without the lists too, so a forest does without them where
    // they find no room
    const size_t pairs = (size_t)max_bg * (size_t)n_trees;
    F->reach_rows = (int)std::min<size_t>(kReachMax, kReachBytes / (pairs * sizeof(Reach)));
    if (F->reach_rows >= kReachMin) {
      const size_t lists = pairs * F->reach_rows * sizeof(Reach);
      if (hipMalloc((void**)&F->reach, lists + (pairs + 1) * sizeof(int32_t)) == hipSuccess) {
        F->reach_cnt = reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(F->reach) + lists);
      } else {
        F->reach = nullptr;
        (void)hipGetLastError();
      }
    }
  }
  if (e != hipSuccess) {
    return ffail(e == hipErrorOutOfMemory ? FSI_ERR_OUT_OF_MEMORY : FSI_ERR_HIP,
                 std::string("forest upload: ") + hipGetErrorString(e));
  }
  guard.f = nullptr;
  *out = F;
  return FSI_OK;
  FSI_ABI_CATCH
}

fsi_status fsi_forest_destroy(fsi_forest_t forest) {
  FSI_ABI_TRY
  free_forest(forest);
  return FSI_OK;
  FSI_ABI_CATCH
}

fsi_status fsi_forest_values(fsi_forest_t F, const double* x_dev, int n_bg, const double* bg_dev,
                             int dtype, void* v_dev, hipStream_t stream) {
  FSI_ABI_TRY
  if (!F) return ffail(FSI_ERR_INVALID_ARG, "forest is NULL");
  if (!x_dev || !bg_dev || !v_dev) return ffail(FSI_ERR_INVALID_ARG, "null device pointer");
  if (n_bg < 1 || n_bg > F->max_bg)
    return ffail(FSI_ERR_INVALID_ARG, "need 1 <= n_bg <= the forest's max_bg");
  if (dtype != FSI_DTYPE_F64 && dtype != FSI_DTYPE_F32)
    return ffail(FSI_ERR_INVALID_ARG, "dtype must be FSI_DTYPE_F64 or FSI_DTYPE_F32");
  if (((uintptr_t)v_dev | (uintptr_t)x_dev | (uintptr_t)bg_dev) & 15u)
    return ffail(FSI_ERR_INVALID_ARG, "device pointers must be 16-byte aligned");
  const int n_chunks = (n_bg + kBgChunk - 1) / kBgChunk;
  const int64_t prep_total = (int64_t)n_chunks * F->n_nodes;
  const int prep_grid = (int)std::min<int64_t>((prep_total + kThreads - 1) / kThreads, 4096);
  const int64_t pairs = (int64_t)n_bg * F->n_trees;
  const bool plain = walk_plain(F->d, pairs, F->depth);
  const int kp = walk_kp(F->d, pairs);
  int32_t* over = F->reach && !plain ? F->reach_cnt + pairs : nullptr;
  prep_kernel<<<prep_grid, kThreads, 0, stream>>>(F->feature, F->threshold, F->left, F->right,
                                                  F->n_nodes, F->d, x_dev, bg_dev, n_bg, F->prep, over);
  ReachLists reach{nullptr, nullptr, nullptr, 0};
  if (F->reach && !plain) {
    const int grid = (int)std::min<int64_t>((pairs + kThreads / 64 - 1) / (kThreads / 64), 4096);
    reach_kernel<<<grid, kThreads, 0, stream>>>(F->prep, F->value, F->roots, F->n_trees, F->n_nodes,
                                                pairs, walk_bits(F->d, kp), F->reach_rows, F->reach, F->reach_cnt, over);
    reach = ReachLists{F->reach, F->reach_cnt, over, F->reach_rows};
  }
  if (dtype == FSI_DTYPE_F64)
    launch_walk(F->prep, F->value, F->roots, F->n_trees, F->n_nodes, F->depth, reach, plain, kp, n_bg,
                F->d, (double*)v_dev, stream);
  else
    launch_walk(F->prep, F->value, F->roots, F->n_trees, F->n_nodes, F->depth, reach, plain, kp, n_bg,
                F->d, (float*)v_dev, stream);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return ffail(FSI_ERR_HIP, std::string("forest launch: ") + hipGetErrorString(e));
  return FSI_OK;
  FSI_ABI_CATCH
}

fsi_status fsi_forest_mobius(fsi_forest_t F, const double* x_dev, int n_bg, const double* bg_dev,
                             double* a_dev, hipStream_t stream) {
  FSI_ABI_TRY
  if (!F) return ffail(FSI_ERR_INVALID_ARG, "forest is NULL");
  if (!x_dev || !bg_dev || !a_dev) return ffail(FSI_ERR_INVALID_ARG, "null device pointer");
  if (n_bg < 1 || n_bg > F->max_bg)
    return ffail(FSI_ERR_INVALID_ARG, "need 1 <= n_bg <= the forest's max_bg");
  if (((uintptr_t)a_dev | (uintptr_t)x_dev | (uintptr_t)bg_dev) & 15u)
    return ffail(FSI_ERR_INVALID_ARG, "device pointers must be 16-byte aligned");
  if (F->n_paths < 0)
    return ffail(FSI_ERR_UNSUPPORTED, "the Moebius route needs at most 2^26 root-to-leaf paths "
                                      "of at most 24 splits (or d <= 24)");
  const int64_t n2 = (int64_t)1 << (F->d - 1);
  fill_kernel<<<(int)std::min<int64_t>((n2 + 4 * kThreads - 1) / (4 * kThreads), 2048), kThreads, 0,
                stream>>>(reinterpret_cast<double2*>(a_dev), n2);
  const int chunks = (F->n_paths + kThreads - 1) / kThreads;
  const int per = scatter_bg(n_bg, chunks);
  const int64_t work = (int64_t)((n_bg + per - 1) / per) * chunks;
  mobius_scatter_kernel<<<(int)std::min<int64_t>(work, kScatterGrid), kThreads, 0, stream>>>(
      F->path_off, F->steps, F->path_leaf, F->n_paths, F->feature, F->threshold, F->value, F->d,
      x_dev, bg_dev, n_bg, per, a_dev);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return ffail(FSI_ERR_HIP, std::string("forest launch: ") + hipGetErrorString(e));
  return FSI_OK;
  FSI_ABI_CATCH
}

fsi_status fsi_forest_values_mobius(fsi_forest_t F, const double* x_dev, int n_bg,
                                    const double* bg_dev, double* work_dev, int dtype,
                                    void* v_dev, hipStream_t stream) {
  FSI_ABI_TRY
  if (!F) return ffail(FSI_ERR_INVALID_ARG, "forest is NULL");
  if (!v_dev) return ffail(FSI_ERR_INVALID_ARG, "null device pointer");
  if (dtype != FSI_DTYPE_F64 && dtype != FSI_DTYPE_F32)
    return ffail(FSI_ERR_INVALID_ARG, "dtype must be FSI_DTYPE_F64 or FSI_DTYPE_F32");
  if ((uintptr_t)v_dev & 15u) return ffail(FSI_ERR_INVALID_ARG, "device pointers must be 16-byte aligned");
  if (dtype == FSI_DTYPE_F32 && (void*)work_dev == v_dev)
    return ffail(FSI_ERR_INVALID_ARG, "an FP32 output needs its own FP64 workspace");
  fsi_status st = fsi_forest_mobius(F, x_dev, n_bg, bg_dev, work_dev, stream);
  if (st != FSI_OK) return st;
  if (dtype == FSI_DTYPE_F32)
    launch_zeta<float>(work_dev, F->d, (float*)v_dev, stream);
  else
    launch_zeta<double>(work_dev, F->d, (double*)v_dev, stream);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return ffail(FSI_ERR_HIP, std::string("forest launch: ") + hipGetErrorString(e));
  return FSI_OK;
  FSI_ABI_CATCH
}

}  // extern "C"
