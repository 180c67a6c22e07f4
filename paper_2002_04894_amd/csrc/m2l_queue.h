// Work queue (and small helpers) of the M2L kernels whose waves each take a target box at a time
// (m2l_lane.hip, m2l_quad.hip).
//
// The targets are ordered with the eight children of a parent side by side,
// parents by decreasing weak-list length in coarse steps (lists.hip), so
// neighbours in the order mostly are neighbours in space and share most of
// their sources.  The order is dealt to the eight XCDs in runs: the waves of
// one XCD work on neighbouring targets at the same time and find each other's
// source expansions in its L2.  A wave whose XCD's runs are used up takes
// targets of the next XCD's.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fmm {
namespace m2lq {

constexpr int kXcds = 8;  // blocks are dispatched to the XCDs in turn

// targets per run: as many as an XCD has waves at work, or one parent's
// children when there are few targets
inline int run_length(int64_t ntarget) { return ntarget >= 32768 ? 256 : 8; }

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

struct Cursor {
  int skip = 0;  // queues found empty, from the home XCD's on
};

// position in the order of the wave's next target, -1 when all are taken;
// called by whole waves
__device__ __forceinline__ int64_t next(Cursor& c, int* __restrict__ queue, int64_t ntarget, int run, int lane) {
  for (; c.skip < kXcds; ++c.skip) {
    const int x = (blockIdx.x + c.skip) % kXcds;
    int k = 0;
    if (lane == 0) k = atomicAdd(&queue[x], 1);
    k = uniform(k);
    const int64_t pos = (int64_t)(k / run) * (kXcds * run) + x * run + k % run;
    if (pos < ntarget) return pos;
  }
  return -1;
}

}  // namespace m2lq
}  // namespace fmm
