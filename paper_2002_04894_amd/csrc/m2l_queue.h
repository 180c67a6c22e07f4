// Work queue and small helpers of the M2L kernels (m2l_lane.hip,
// m2l_quad.hip), whose waves each take a target box at a time, or whose blocks
// share one target out among their waves.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fmm_internal.h"

namespace fmm {
namespace m2lq {

constexpr int kXcds = 8;   // blocks are dispatched to the XCDs in turn
constexpr int kRun = 256;  // targets per run: as many as an XCD has waves at work

// a value that is the same in all lanes, in scalar registers
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// 1/sqrt(x), 0 for x = 0: the hardware estimate and two Newton steps
__device__ __forceinline__ double rsqrt0(double x) {
  double y = x > 0.0 ? __builtin_amdgcn_rsq(x) : 0.0;
  const double h = 0.5 * x;
  y = y * (1.5 - h * y * y);
  return y * (1.5 - h * y * y);
}

// N values of a lane: in LDS words of its own (the words of neighbouring lanes
// side by side, `stride` apart) or, with LDS = false, in registers.  Values
// that would spill are parked in LDS: spilled to scratch memory they would have
// to come back through an L2 that the gathered expansions have swept (31
// spilled registers made the binary64 kernel's launch 1.4 times as long at
// order 12).
template <class T, int N, bool LDS>
struct Kept {
  T* w;
  int stride;
  T v[LDS ? 1 : N];
  __device__ __forceinline__ Kept(T* words, int st) : w(words), stride(st) {}
  __device__ __forceinline__ void put(int i, T x) {
    if constexpr (LDS)
      w[i * stride] = x;
    else
      v[i] = x;
  }
  __device__ __forceinline__ T get(int i) const {
    if constexpr (LDS) {
      asm volatile("" ::: "memory");  // read back, not kept in a register since put()
      return w[i * stride];
    } else {
      return v[i];
    }
  }
};

// How a launch deals out its targets.  Persistent waves take one target each
// (Cursor below); or, with SHARE, block b takes the target at position b, and
// its waves take the batches of the list in turn: with few targets (trees of
// up to three levels) most waves would have nothing to do, and a list longer
// than a wave's share of the launch would hold it up.  The waves of a block
// are kept together and wait for memory at the same time, so with more targets
// this costs the binary64 kernel, one block of eight waves to a CU, more than
// it gives, except for the lists that are too long; the per-lane kernel, up to
// four blocks of four waves to a CU, gains up to kShareLane targets.
// Measured, M2L in us (waves by themselves / SHARE): binary64 order 12, 47,003
// points on a sphere, 512 leaves 545 / 150; 2^18 Plummer points, 4,096 leaves
// 4,240 / 6,000; 200,000 points on a sphere, 4,096 leaves 3,730 / 1,960 with the
// long lists shared; binary32 order 6, 200,000 points, 4,096 leaves 350 / 215.
// The numbers of targets are 8, 72, 584, 4,680, 37,448, 299,592, ...: the limits
// mean trees of up to three levels, of up to four and, for kM2LSiblingsMin, of
// six and more; what was measured are the numbers on their two sides.
constexpr int64_t kShareQuad = 1024;  // all targets shared up to here,
constexpr int64_t kShareLane = 8192;  // and up to here (per-lane kernel)
constexpr int64_t kLongQuad = 8192;   // binary64: the too long ones up to here

// The waves' next targets.  With siblings side by side in the order (RUNS) it
// is dealt to the XCDs in runs, so that the waves of one XCD work on
// neighbours at the same time and find each other's source expansions in its
// L2; else one counter serves all.
template <bool RUNS>
struct Cursor {
  int x = RUNS ? blockIdx.x % kXcds : 0;  // the counter it takes from
  __device__ __forceinline__ static int64_t position(int c, int k) {
    return RUNS ? (int64_t)(k / kRun) * (kXcds * kRun) + c * kRun + k % kRun : k;
  }
  // position in the order, ntarget or more when all targets are taken
  __device__ __forceinline__ int64_t next(int* __restrict__ queue, int64_t ntarget, int lane) {
    for (;;) {
      int k = 0;
      if (lane == 0) k = atomicAdd(&queue[x], 1);
      const int64_t pos = position(x, uniform(k));
      if (!RUNS || pos < ntarget) return pos;
      // used up: the next counter that is not, by one look at all of them
      const int v = __hip_atomic_load(&queue[lane % kXcds], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t left = (uint32_t)__ballot(position(lane % kXcds, v) < ntarget) & 0xffu;
      if (left == 0) return ntarget;
      x = (x + __ffs((int)((left >> x) | (left << (kXcds - x)))) - 1) % kXcds;
    }
  }
};

}  // namespace m2lq
}  // namespace fmm
