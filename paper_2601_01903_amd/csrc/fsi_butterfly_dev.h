// Device code of the whole-vector butterflies: the Moebius transform
// (fsi_kernels.hip) and the subset sums of the value functions
// (fsi_forest.hip).
//
// One pass of a butterfly (Moebius transform or subset sums) over the G bits
// [lo, lo + G) of one vector. A work item is a tile of 2^kMobTileBits elements: 2^cb consecutive low
// indices (cb = kMobTileBits - G; 0 for the low pass, lo = 0) for each
// setting of the G bits, at one setting of the other bits. A thread holds 16
// elements of the tile, i.e. four of its bits, in registers, runs those
// levels there and hands the tile to the next four through LDS, so a pass
// reads and writes each value once with one exchange for G <= 8 and three for
// the low pass. (One level per LDS round trip and barrier, as before, held a
// pass over 2^24 FP64 values at 64 us where memory allows 40.)
//
// Every layout is an affine map of the thread: mob_field(t, P) | k << P puts
// the four register bits k at tile bits P .. P + 3. Global accesses use
// P >= 4, whose waves touch runs of at least 16 consecutive elements. The
// levels run in ascending order of their bits.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "fsi_kernels.h"

namespace fsi {

constexpr int kMobElems = 16;                       // per thread
constexpr int kMobThreads = (1 << kMobTileBits) / kMobElems;

// LDS place of tile element e: one element of padding per 16, so that lanes
// 16 and 256 elements apart meet different banks.
__device__ __forceinline__ int mob_pad(int e) { return e + (e >> 4); }
constexpr int kMobLds = (1 << kMobTileBits) + (1 << kMobTileBits >> 4);
__device__ __forceinline__ int mob_field(int t, int p) {
  return (t & ((1 << p) - 1)) | ((t >> p) << (p + 4));
}
// levels [j0, 4) of the four register bits: each element with the bit set
// becomes Op::op(itself, its partner without the bit)
template <typename Op, typename T>
__device__ __forceinline__ void mob_levels(T (&x)[kMobElems], int j0) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j >= j0) {
#pragma unroll
      for (int k = 0; k < kMobElems; ++k)
        if (k & (1 << j)) x[k] = Op::op(x[k], x[k ^ (1 << j)]);
    }
}
// the tile from layout `from` to layout `to`
template <typename T>
__device__ __forceinline__ void mob_exchange(T* m, T (&x)[kMobElems], int from, int to) {
  const int a = mob_field(threadIdx.x, from), b = mob_field(threadIdx.x, to);
#pragma unroll
  for (int k = 0; k < kMobElems; ++k) m[mob_pad(a | (k << from))] = x[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kMobElems; ++k) x[k] = m[mob_pad(b | (k << to))];
  __syncthreads();
}

// Element e of a high pass's tile, from the tile's first element: 2^cb
// consecutive elements for each setting of the group bits above them.
__device__ __forceinline__ int64_t mob_high_at(int e, int cb, int lo) {
  return ((int64_t)(e >> cb) << lo) + (e & ((1 << cb) - 1));
}

}  // namespace fsi
