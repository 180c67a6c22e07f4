// Near field (P2P, Algorithm 4) and the evaluation driver (Algorithm 1:
// P2M, M2M; Algorithm 3: M2L, L2L; Algorithm 4: L2P, P2P).
//
// P2P: for every target point t of leaf i and every source s of a leaf j
// strongly connected to i (i itself included), phi_t += q_s / r and
// E_t += q_s (x_t - x_s) / r^3, skipping pairs at distance 0 (this removes
// the self term j = i of eq. (2.1)).  Each target pulls from its full list
// (gather form: no atomics, deterministic).  On clustered data the strong
// lists of a few leaves hold far more sources than the rest, so each list is
// cut into segments of about kP2PSeg source points (a plan made once per
// tree); one workgroup takes one segment.  A leaf with one segment
// writes its result directly; the segments of a split leaf write partial sums
// that a second pass adds up in segment order.
#include <algorithm>
#include <type_traits>

#include "fmm_internal.h"
#include "lane_ops.h"
#include "launch_rules.h"
#include "tile_layout.h"

namespace fmm {

void launch_p2m(const Tree& t, const Tables& tb, const double* qt, double* Mx, hipStream_t s);
void launch_m2m(const Tree& t, int l, const Tables& tb, double* Mx, hipStream_t s);
void launch_m2l(const Tree& t, const Tables& tb, const double* Mx, double* Lx, int prec, hipStream_t s);
void launch_l2l(const Tree& t, int l, const Tables& tb, double* Lx, hipStream_t s);
void launch_l2p(const Tree& t, const Tables& tb, const double* Lx, const int32_t* start, const double* px,
                const double* py, const double* pz, double* f0, double* f1, double* f2, double* f3, hipStream_t s);

namespace {

__global__ void k_gather(const double* __restrict__ q, const int32_t* __restrict__ perm, double* __restrict__ qt,
                         int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) qt[i] = q[perm[i]];
}

// 1/sqrt(r2) to full double precision: hardware estimate + one Newton step
// (relative error below 5e-15); 0 for r2 == 0.  The estimate of +0 is +inf,
// whose low word is zero, so clearing its high word gives +0 and the Newton
// step then keeps 0: one select of one word instead of two on the result.
__device__ __forceinline__ double rsqrt_nr(double r2) {
  const double e = __builtin_amdgcn_rsq(r2);
  const long long b = __double_as_longlong(e);
  const int hi = r2 > 0.0 ? (int)(b >> 32) : 0;
  const double y0 = __hiloint2double(hi, (int)b);
  return y0 * (1.5 - 0.5 * r2 * y0 * y0);
}

// Work items (segments, in leaf order) are mapped to blocks so that
// consecutive ones, whose sources overlap, run on the same XCD and share its
// L2.
__device__ __forceinline__ int64_t xcd_leaf(int64_t nleaf) {
  const int64_t per = (nleaf + 7) / 8;
  return (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
}

constexpr int kP2PBuf = 256;     // source points staged per chunk (x, y, z, q): 8 KB of LDS, 3 waves per SIMD
constexpr int64_t kP2PSeg = 8192;  // source points per work item (about)

// ---- the plan: one wave per leaf walks its strong list 64 entries at a
// time.  Entry e starts a segment when it is the first of the list or when
// floor(sources before e / kP2PSeg) changes at e.
__device__ __forceinline__ int64_t wave_incl_scan64(int64_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t t = __shfl_up(v, d);
    if (lane >= d) v += t;
  }
  return v;
}

template <bool FILL>
__global__ __launch_bounds__(256) void k_seg_plan(int64_t nleaf, const int32_t* __restrict__ start,
                                                  const int64_t* __restrict__ s_off, const int32_t* __restrict__ s_idx,
                                                  int32_t* __restrict__ nseg, int64_t* __restrict__ work,
                                                  const int64_t* __restrict__ leaf_seg, int32_t* __restrict__ seg_leaf,
                                                  int64_t* __restrict__ seg_e0) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= nleaf) return;
  const int64_t e0 = s_off[i], e1 = s_off[i + 1];
  const uint64_t below = (1ull << lane) - 1ull;
  int64_t carry = 0;  // sources of the entries before this chunk
  int prev_last = 0;  // sources of the entry just before this chunk
  int64_t flags = 0;  // segments started so far
  const int64_t base = FILL ? leaf_seg[i] : 0;
  for (int64_t k0 = e0; k0 < e1; k0 += 64) {
    const int64_t e = k0 + lane;
    const bool valid = e < e1;
    int cnt = 0;
    if (valid) {
      const int j = s_idx[e];
      cnt = start[j + 1] - start[j];
    }
    const int64_t incl = wave_incl_scan64(cnt, lane);
    const int64_t excl = carry + incl - cnt;
    const int up = __shfl_up(cnt, 1);
    const int prev = lane == 0 ? prev_last : up;
    const bool flag = valid && (e == e0 || excl / kP2PSeg != (excl - prev) / kP2PSeg);
    const uint64_t m = __ballot(flag);
    if (FILL && flag) {
      const int64_t pos = base + flags + __popcll(m & below);
      seg_leaf[pos] = (int32_t)i;
      seg_e0[pos] = e;
    }
    flags += __popcll(m);
    carry += __shfl(incl, 63);
    prev_last = __shfl(cnt, 63);
  }
  if (!FILL && lane == 0) {
    nseg[i] = (int32_t)flags;
    work[i] = (int64_t)(start[i + 1] - start[i]) * carry;  // interactions of this leaf
  }
}

// partial sums needed by leaf i: one per target and segment when split
__global__ void k_part_count(int64_t nleaf, const int32_t* __restrict__ start, const int32_t* __restrict__ nseg,
                             int64_t* __restrict__ cnt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nleaf) cnt[i] = nseg[i] > 1 ? (int64_t)nseg[i] * (start[i + 1] - start[i]) : 0;
}

__global__ void k_sum64(int64_t n, const int64_t* __restrict__ v, unsigned long long* __restrict__ acc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long x = i < n ? (unsigned long long)v[i] : 0ull;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
  if ((threadIdx.x & 63) == 0) atomicAdd(acc, x);
}

// One workgroup of W waves per segment.  A wave's lanes hold T targets each (tl,
// tl + TT, ...) and one of R source streams, R TT <= 64, so every source read
// from LDS serves T interactions.  Sources are staged in chunks of up to
// kP2PBuf points gathered from consecutive entries of the segment: the lanes
// take the chunk's points in a flat order, so all their loads are in flight
// together.  The targets of leaf b are [tstart[b], tstart[b+1]) of (tx, ty,
// tz), written to index tperm[.] of the outputs: the leaf's own sources
// (tstart = start, tx = px, tperm = perm) or the separate targets grouped by
// leaf.
// Binary64: T, TT and R by the number of targets (p2p_split), and the waves take
// contiguous parts of the segment's entries.
// Binary32 near field (F32): coordinates are taken relative to the target
// leaf's cell centre in binary64 and rounded to binary32, so that the
// differences of nearby points keep binary32 accuracy; 1/r is the hardware
// binary32 reciprocal square root; each lane sums the interactions of one
// staged chunk in binary32 and adds the chunk sums into compensated binary32
// accumulators (Kahan); the results are widened to binary64 before the far field
// is added.  The chunks, a lane's share of them and the order of their sums are
// the same for every W, as they fix the binary32 roundings: the waves take the
// chunks in turn, and the chunk sums of a round meet in LDS, where every wave
// adds up some of the accumulators in chunk order.  Two distinct points whose relative coordinates round to the same
// binary32 values count as coincident (contribute nothing).
struct Kahan {
  float s = 0.f, c = 0.f;
  __device__ __forceinline__ void add(float v) {
    const float y = v - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
  }
  __device__ __forceinline__ double get() const { return (double)s - (double)c; }
};

// Orders a wave's LDS accesses around a point (other lanes of the wave read
// what this lane wrote): the LDS unit executes a wave's instructions in order.
__device__ __forceinline__ void p2p_wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The near field of one segment: its entries, in LDS as far as they fit
// (kP2PEntries: the first point of the source leaf, its points), so that a
// chunk waits for its points only and not for two loads before them.
constexpr int kP2PEntries = 512;
constexpr int kP2PSlots = 2;  // binary32: chunks of a wave in a round
struct P2PSeg {
  const int32_t* s_idx;  // the segment's first entry
  const int32_t* start;
  int ne;                // entries
  const int32_t* base;   // LDS
  const int32_t* cnt;
  __device__ __forceinline__ void entry(int i, int& b, int& n) const {
    if (i < kP2PEntries) {
      b = base[i];
      n = cnt[i];
    } else {
      const int j = s_idx[i];
      b = start[j];
      n = start[j + 1] - b;
    }
  }
};

// Stages the next chunk of entries [e, e1) (off: points of entry e staged
// before) into buf, moves (e, off) past it and returns its points; with STAGE
// false only moves on.
template <bool F32, bool STAGE, class V>
__device__ __forceinline__ int p2p_chunk(const P2PSeg& sg, int e1, int& e, int& off, V* buf, int lane,
                                         const double* __restrict__ px, const double* __restrict__ py,
                                         const double* __restrict__ pz, const double* __restrict__ qt, double ccx,
                                         double ccy, double ccz) {
  // up to 16 entries from e on: lane q < 16 takes entry e + q
  int base = 0, cnt = 0;
  if (lane < 16 && e + lane < e1) {
    sg.entry(e + lane, base, cnt);
    if (lane == 0) {
      base += off;
      cnt -= off;
    }
  }
  int pre = cnt;  // inclusive prefix over lanes 0..15
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
    const int v = __shfl_up(pre, d, 16);
    if ((lane & 15) >= d) pre += v;
  }
  const int all = __shfl(pre, 15);
  const int fill = all < kP2PBuf ? all : kP2PBuf;
  const int avail = e1 - e < 16 ? e1 - e : 16;
  if constexpr (STAGE) {
    // flat point f of the chunk lies in entry q: pre[q-1] <= f < pre[q];
    // all loads of the chunk are issued before the LDS stores
    constexpr int kIt = kP2PBuf / 64;
    double4 v[kIt];
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
      const int f = it * 64 + lane;
      int q = 0;
#pragma unroll
      for (int k = 0; k < 15; ++k) q += (__shfl(pre, k) <= f) ? 1 : 0;
      const int lo = __shfl(pre, q) - __shfl(cnt, q);
      const int u = __shfl(base, q) + (f - lo);
      if (f < fill) v[it] = make_double4(px[u], py[u], pz[u], qt[u]);
    }
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
      const int f = it * 64 + lane;
      if (f < fill) {
        if constexpr (F32)
          buf[f] = make_float4((float)(v[it].x - ccx), (float)(v[it].y - ccy), (float)(v[it].z - ccz), (float)v[it].w);
        else
          buf[f] = v[it];
      }
    }
  }
  // entries staged completely, and how far into the next one
  const int done = __popcll(__ballot(lane < avail && pre <= fill));
  if (done < avail) {
    const int prev = done == 0 ? 0 : __shfl(pre, done - 1);
    off = (done == 0 ? off : 0) + (fill - prev);
  } else {
    off = 0;
  }
  e += done;
  return fill;
}

// Targets per lane T (1 .. 4), lanes per target row TT and source streams R of a
// leaf with nt targets in binary64: the T of least time per source, T / R, the
// largest on ties (fewer LDS reads).  Two targets per lane and powers of two
// for TT left a third of the lanes idle at 39 targets (20,000 points, 512
// leaves: T 4, TT 10, R 6) and a quarter at 92.
struct P2PSplit {
  int T, TT, R;
};
__device__ __forceinline__ P2PSplit p2p_split(int nt) {
  P2PSplit best{1, nt < 64 ? (nt > 0 ? nt : 1) : 64, 1};
  best.R = 64 / best.TT;
  int rows = (nt + 63) / 64;
  // cost T / R, times the passes over the sources; compared as fractions
#pragma unroll
  for (int T = 2; T <= 4; ++T) {
    int tt = (nt + T - 1) / T;
    tt = tt < 1 ? 1 : tt > 64 ? 64 : tt;
    const int r = 64 / tt, pass = (nt + T * tt - 1) / (T * tt);
    if (T * pass * best.R <= best.T * rows * r) {
      best = P2PSplit{T, tt, r};
      rows = pass;
    }
  }
  return best;
}

struct P2POut {
  double4* part;  // partial sums by target - t0, or null: then the far field is
                  // added and the results go to the outputs
  const double *f0, *f1, *f2, *f3;
  const int32_t* perm;
  double *pot, *ex, *ey, *ez;
  __device__ __forceinline__ void put(int t, int t0, double f, double gx, double gy, double gz) const {
    if (part) {
      part[t - t0] = make_double4(f, gx, gy, gz);
      return;
    }
    if (f0) {
      f += f0[t];
      gx += f1[t];
      gy += f2[t];
      gz += f3[t];
    }
    const int o = perm[t];
    pot[o] = f;
    ex[o] = gx;
    ey[o] = gy;
    ez[o] = gz;
  }
};

// The targets [t0, t1) of a leaf against the segment, T TT of them per pass, the
// passes dealt to the blocks in y (the same sums as in one block); red: 4 T W 64 doubles of
// LDS for the sums of the waves (W > 1; it may be the waves' buffers).
template <bool F32, int T, int W, class V>
__device__ __forceinline__ void p2p_targets(const P2PSeg& sg, int t0, int t1, int TT, int R, V* buf, double* red,
                                            const double* __restrict__ px, const double* __restrict__ py,
                                            const double* __restrict__ pz, const double* __restrict__ qt,
                                            const double* __restrict__ tx, const double* __restrict__ ty,
                                            const double* __restrict__ tz, double ccx, double ccy, double ccz,
                                            const P2POut& out) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int tl = lane % TT, h = lane / TT;
  const bool lane_on = h < R;
  // positions are unsigned: past the last target they may exceed 2^31
  for (unsigned c0 = t0 + blockIdx.y * T * TT; c0 < (unsigned)t1; c0 += gridDim.y * T * TT) {
    double f[T][4] = {};
    double x[T], y[T], z[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const unsigned t = c0 + tl + i * TT, u = t < (unsigned)t1 ? t : t0;
      x[i] = tx[u];
      y[i] = ty[u];
      z[i] = tz[u];
    }
    // this wave's entries
    int e = F32 ? 0 : (int)((int64_t)sg.ne * w / W), off = 0;
    const int e1 = F32 ? sg.ne : (int)((int64_t)sg.ne * (w + 1) / W);
    if constexpr (F32) {
      float xf[T], yf[T], zf[T], s[T][4] = {};
#pragma unroll
      for (int i = 0; i < T; ++i) {
        xf[i] = (float)(x[i] - ccx);
        yf[i] = (float)(y[i] - ccy);
        zf[i] = (float)(z[i] - ccz);
      }
      auto interact = [&](const float4 v) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
          const float dx = xf[i] - v.x, dy = yf[i] - v.y, dz = zf[i] - v.z;
          const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dx, dx, dy * dy));
          const float inv = r2 > 0.f ? __builtin_amdgcn_rsqf(r2) : 0.f;
          const float qi = v.w * inv;
          const float qi3 = qi * inv * inv;
          s[i][0] = __builtin_fmaf(v.w, inv, s[i][0]);
          s[i][1] = __builtin_fmaf(qi3, dx, s[i][1]);
          s[i][2] = __builtin_fmaf(qi3, dy, s[i][2]);
          s[i][3] = __builtin_fmaf(qi3, dz, s[i][3]);
        }
      };
      // the sums of the next chunk, in s
      auto chunk = [&] {
        const int fill = p2p_chunk<F32, true>(sg, e1, e, off, buf, lane, px, py, pz, qt, ccx, ccy, ccz);
        p2p_wave_fence();
        int u = h;
        for (; u + 3 * R < fill; u += 4 * R) {
          const float4 s0 = buf[u], s1 = buf[u + R], s2 = buf[u + 2 * R], s3 = buf[u + 3 * R];
          interact(s0);
          interact(s1);
          interact(s2);
          interact(s3);
        }
        for (; u < fill; u += R) interact(buf[u]);
        p2p_wave_fence();
      };
      if constexpr (W == 1) {
        Kahan k[T][4];
        while (e < e1) {
          chunk();
#pragma unroll
          for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              k[i][j].add(s[i][j]);
              s[i][j] = 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) f[i][j] = k[i][j].get();
      } else {
        constexpr int NQ = T * 4 / W;  // accumulators of a wave: w, w + W, ...
        static_assert(NQ * W == T * 4, "");
        float* cs = (float*)red;       // [slot][accumulator][lane]
        Kahan k[NQ];
        while (e < e1) {
          int slot = 0;
          for (; slot < kP2PSlots * W && e < e1; ++slot) {
            if (slot % W != w) {
              p2p_chunk<F32, false>(sg, e1, e, off, buf, lane, px, py, pz, qt, ccx, ccy, ccz);
              continue;
            }
            chunk();
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                cs[(slot * T * 4 + i * 4 + j) * 64 + lane] = s[i][j];
                s[i][j] = 0.f;
              }
          }
          __syncthreads();
          for (int c = 0; c < slot; ++c)
#pragma unroll
            for (int i = 0; i < NQ; ++i) k[i].add(cs[(c * T * 4 + w + i * W) * 64 + lane]);
          __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) red[(w + i * W) * 64 + lane] = k[i].get();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) f[i][j] = red[(i * 4 + j) * 64 + lane];
      }
    } else {
      auto interact = [&](const double4 v) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
          const double dx = x[i] - v.x, dy = y[i] - v.y, dz = z[i] - v.z;
          const double inv = rsqrt_nr(dx * dx + dy * dy + dz * dz);
          const double qi = v.w * inv;
          const double qi3 = qi * inv * inv;
          f[i][0] += qi;
          f[i][1] += qi3 * dx;
          f[i][2] += qi3 * dy;
          f[i][3] += qi3 * dz;
        }
      };
      while (e < e1) {
        const int fill = p2p_chunk<F32, true>(sg, e1, e, off, buf, lane, px, py, pz, qt, ccx, ccy, ccz);
        p2p_wave_fence();
        int u = lane_on ? h : fill;
        for (; u + R < fill; u += 2 * R) {
          const double4 s0 = buf[u], s1 = buf[u + R];
          interact(s0);
          interact(s1);
        }
        for (; u < fill; u += R) interact(buf[u]);
        p2p_wave_fence();
      }
    }
    // sum the source streams (fixed order): binary32 has powers of two and
    // halves them, as for any W
    if constexpr (F32) {
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        if (d >= TT) {
#pragma unroll
          for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) f[i][j] += __shfl_xor(f[i][j], d);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double v = f[i][j];
          for (int r = 1; r < R; ++r) f[i][j] += __shfl(v, tl + r * TT);
        }
    }
    if constexpr (!F32 && W > 1) {  // the waves' sums, in wave order
      __syncthreads();
      if (w > 0 && lane < TT)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) red[((w - 1) * T * 4 + i * 4 + j) * 64 + lane] = f[i][j];
      __syncthreads();
      if (w == 0 && lane < TT)
        for (int v = 0; v < W - 1; ++v)
#pragma unroll
          for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) f[i][j] += red[(v * T * 4 + i * 4 + j) * 64 + lane];
    }
    if (w == 0 && lane < TT) {
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const unsigned t = c0 + tl + i * TT;
        if (t < (unsigned)t1) out.put((int)t, t0, f[i][0], f[i][1], f[i][2], f[i][3]);
      }
    }
    if constexpr (W > 1) __syncthreads();  // red read before the buffers are filled again
  }
}

template <bool F32, int W>
__global__ __launch_bounds__(64 * W) void k_p2p(
    int64_t nseg, const int32_t* __restrict__ seg_leaf, const int64_t* __restrict__ seg_e0,
    const int64_t* __restrict__ leaf_seg, const int64_t* __restrict__ leaf_part, const int32_t* __restrict__ start,
    const int64_t* __restrict__ s_off, const int32_t* __restrict__ s_idx, const double* __restrict__ px,
    const double* __restrict__ py, const double* __restrict__ pz, const double* __restrict__ qt,
    const int32_t* __restrict__ tstart, const double* __restrict__ tx, const double* __restrict__ ty,
    const double* __restrict__ tz, const int32_t* __restrict__ perm, const double* __restrict__ f0,
    const double* __restrict__ f1, const double* __restrict__ f2, const double* __restrict__ f3,
    double4* __restrict__ part, double* __restrict__ pot, double* __restrict__ ex, double* __restrict__ ey,
    double* __restrict__ ez, const double* __restrict__ lgeom) {
  typedef typename std::conditional<F32, float4, double4>::type V;
  // the waves' chunks (8 KB each, 4 KB in binary32); in binary64 later their
  // sums, at most 4 x 4 x 64 doubles a wave
  constexpr int kBytes = (int)sizeof(V) * kP2PBuf;
  static_assert(F32 || kBytes >= 4 * 4 * 64 * 8, "");
  constexpr int kSums = F32 && W > 1 ? kP2PSlots * W * 2 * 4 * 64 * 4 : 0;  // binary32: the chunk sums of a round
  __shared__ __align__(16) char lds[W * kBytes + kSums];
  __shared__ int32_t ebase[kP2PEntries], ecnt[kP2PEntries];
  const int64_t g = xcd_leaf(nseg);
  if (g >= nseg) return;
  const int64_t b = seg_leaf[g];
  const int64_t sb = leaf_seg[b], ns = leaf_seg[b + 1] - sb, r = g - sb;
  const int64_t e0 = seg_e0[g], e1 = r + 1 < ns ? seg_e0[g + 1] : s_off[b + 1];
  const int t0 = tstart[b], t1 = tstart[b + 1];
  const int nt = t1 - t0;
  const P2PSplit sp = F32 ? P2PSplit{2, nt <= 16 ? 8 : (nt <= 32 ? 16 : (nt <= 64 ? 32 : 64)), 0} : p2p_split(nt);
  if (blockIdx.y > 0 && (int64_t)blockIdx.y * sp.T * sp.TT >= nt) return;  // no pass left for this block
  const P2PSeg sg{s_idx + e0, start, (int)(e1 - e0), ebase, ecnt};
  for (int i = threadIdx.x; i < sg.ne && i < kP2PEntries; i += 64 * W) {
    const int j = sg.s_idx[i], u = start[j];
    ebase[i] = u;
    ecnt[i] = start[j + 1] - u;
  }
  __syncthreads();
  const P2POut out{ns > 1 ? part + leaf_part[b] + r * nt : nullptr, f0, f1, f2, f3, perm, pot, ex, ey, ez};
  V* buf = (V*)(lds + (threadIdx.x >> 6) * kBytes);
  double* red = (double*)(F32 ? lds + W * kBytes : lds);
  if constexpr (F32) {
    const double ccx = lgeom[b * 10 + 6], ccy = lgeom[b * 10 + 7], ccz = lgeom[b * 10 + 8];
    p2p_targets<true, 2, W>(sg, t0, t1, sp.TT, 64 / sp.TT, buf, red, px, py, pz, qt, tx, ty, tz, ccx, ccy, ccz, out);
  } else {
    auto go = [&](auto t) __attribute__((always_inline)) {
      p2p_targets<false, decltype(t)::value, W>(sg, t0, t1, sp.TT, sp.R, buf, red, px, py, pz, qt, tx, ty, tz, 0.0, 0.0,
                                                0.0, out);
    };
    if (sp.T == 4)
      go(std::integral_constant<int, 4>{});
    else if (sp.T == 3)
      go(std::integral_constant<int, 3>{});
    else if (sp.T == 2)
      go(std::integral_constant<int, 2>{});
    else
      go(std::integral_constant<int, 1>{});
  }
}

// Results of the leaves not written by k_p2p: with partial sums (NEAR = 1)
// the split leaves, their segments added in order; without the near field
// (NEAR = 0) every leaf.  One wave per leaf, lanes over targets.
template <int NEAR>
__global__ __launch_bounds__(256) void k_p2p_final(int64_t nleaf, const int32_t* __restrict__ start,
                                                   const int64_t* __restrict__ leaf_seg,
                                                   const int64_t* __restrict__ leaf_part,
                                                   const double4* __restrict__ part,
                                                   const int32_t* __restrict__ perm, const double* __restrict__ f0,
                                                   const double* __restrict__ f1, const double* __restrict__ f2,
                                                   const double* __restrict__ f3, double* __restrict__ pot,
                                                   double* __restrict__ ex, double* __restrict__ ey,
                                                   double* __restrict__ ez) {
  const int lane = threadIdx.x & 63;
  const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= nleaf) return;
  const int64_t ns = NEAR ? leaf_seg[b + 1] - leaf_seg[b] : 0;
  if (NEAR && ns <= 1) return;
  const int t0 = start[b], t1 = start[b + 1], nt = t1 - t0;
  for (unsigned t = (unsigned)t0 + lane; t < (unsigned)t1; t += 64) {
    double f = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    if (NEAR) {
      const double4* pp = part + leaf_part[b] + (t - t0);
      for (int64_t r = 0; r < ns; ++r) {
        const double4 v = pp[r * nt];
        f += v.x;
        gx += v.y;
        gy += v.z;
        gz += v.w;
      }
    }
    if (f0) {
      f += f0[t];
      gx += f1[t];
      gy += f2[t];
      gz += f3[t];
    }
    const int o = perm[t];
    pot[o] = f;
    ex[o] = gx;
    ey[o] = gy;
    ez[o] = gz;
  }
}

// partial sums needed for the separate targets of leaf i
__global__ void k_tpart_count(int64_t nleaf, const int32_t* __restrict__ tstart, const int64_t* __restrict__ leaf_seg,
                              int64_t* __restrict__ cnt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nleaf) return;
  const int64_t ns = leaf_seg[i + 1] - leaf_seg[i];
  cnt[i] = ns > 1 ? ns * (int64_t)(tstart[i + 1] - tstart[i]) : 0;
}

}  // namespace

void p2p_plan_targets(Tree& t, hipStream_t s) {
  const int64_t nleaf = t.lev[t.L].nbox;
  int64_t* pcnt = (int64_t*)dalloc(nleaf * sizeof(int64_t), s);
  k_tpart_count<<<(unsigned)((nleaf + 255) / 256), 256, 0, s>>>(nleaf, t.tstart, t.p2p_leaf_seg, pcnt);
  HIPCHECK(hipGetLastError());
  t.p2p_leaf_tpart = (int64_t*)dalloc((nleaf + 1) * sizeof(int64_t), s);
  scan_counts(pcnt, t.p2p_leaf_tpart, nleaf, 0, s);
  int64_t* h = host_stage();
  HIPCHECK(hipMemcpyAsync(h, t.p2p_leaf_tpart + nleaf, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  HIPCHECK(hipStreamSynchronize(s));
  t.p2p_ntpart = *h;
  dfree(pcnt, s);
}

void p2p_plan(Tree& t, hipStream_t s) {
  const Level& V = t.lev[t.L];
  const int64_t nleaf = V.nbox;
  int32_t* nseg = (int32_t*)dalloc(nleaf * sizeof(int32_t), s);
  int64_t* work = (int64_t*)dalloc(nleaf * sizeof(int64_t), s);
  const unsigned gw = (unsigned)((nleaf + 3) / 4);
  k_seg_plan<false><<<gw, 256, 0, s>>>(nleaf, V.start, V.s_off, V.s_idx, nseg, work, nullptr, nullptr, nullptr);
  HIPCHECK(hipGetLastError());
  t.p2p_leaf_seg = (int64_t*)dalloc((nleaf + 1) * sizeof(int64_t), s);
  t.p2p_leaf_part = (int64_t*)dalloc((nleaf + 1) * sizeof(int64_t), s);
  int64_t* h = host_stage();
  if (nleaf <= kSmallScan) {
    scan_plan_small(nseg, V.start, work, t.p2p_leaf_seg, t.p2p_leaf_part, nleaf, h, s);
  } else {
    int64_t* pcnt = (int64_t*)dalloc(nleaf * sizeof(int64_t), s);
    unsigned long long* acc = (unsigned long long*)dalloc(sizeof(unsigned long long), s);
    HIPCHECK(hipMemsetAsync(acc, 0, sizeof(unsigned long long), s));
    scan_counts(nseg, t.p2p_leaf_seg, nleaf, 0, s);
    k_part_count<<<(unsigned)((nleaf + 255) / 256), 256, 0, s>>>(nleaf, V.start, nseg, pcnt);
    HIPCHECK(hipGetLastError());
    scan_counts(pcnt, t.p2p_leaf_part, nleaf, 0, s);
    k_sum64<<<(unsigned)((nleaf + 255) / 256), 256, 0, s>>>(nleaf, work, acc);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipMemcpyAsync(&h[0], t.p2p_leaf_seg + nleaf, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIPCHECK(hipMemcpyAsync(&h[1], t.p2p_leaf_part + nleaf, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIPCHECK(hipMemcpyAsync(&h[2], acc, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    dfree(pcnt, s);
    dfree(acc, s);
  }
  HIPCHECK(hipStreamSynchronize(s));
  check_points_flag();
  t.p2p_nseg = h[0];
  t.p2p_npart = h[1];
  t.p2p_pairs = h[2] - t.n;  // minus the n self pairs
  t.p2p_seg_leaf = (int32_t*)dalloc(std::max<int64_t>(1, t.p2p_nseg) * sizeof(int32_t), s);
  t.p2p_seg_e0 = (int64_t*)dalloc(std::max<int64_t>(1, t.p2p_nseg) * sizeof(int64_t), s);
  k_seg_plan<true><<<gw, 256, 0, s>>>(nleaf, V.start, V.s_off, V.s_idx, nullptr, nullptr, t.p2p_leaf_seg,
                                      t.p2p_seg_leaf, t.p2p_seg_e0);
  HIPCHECK(hipGetLastError());
  dfree(nseg, s);
  dfree(work, s);
}

// prec: FMM_PREC_F64; FMM_PREC_MIXED for the binary32 M2L; FMM_PREC_F32 for
// the binary32 M2L and the binary32 near field (k_p2p<true>: its field loses
// up to a few 1e-5 relative on clustered clouds, through the cancellation among
// near contributions, so it serves loose tolerances only)
namespace {

// Upward and downward passes (Algorithm 1: P2M, M2M; Algorithm 3: M2L, L2L)
// for charges qt in tree order, then L2P at the points (px, py, pz) grouped by
// leaf as [start[b], start[b+1]) into far[0..3] (allocated here).
void far_field(const Tree& t, const double* qt, int p, int prec, const int32_t* start, const double* px,
               const double* py, const double* pz, int64_t npts, double* far[4], hipStream_t s) {
  const int L = t.L;
  PhaseTimer& tm = timer();
  const Tables& tb = tables_for(p, s);
  double* Mx = (double*)dalloc((size_t)t.nbox_total * tb.stride * sizeof(double), s);
  // M2L reads its own copy of the multipoles and writes every local expansion
  // of levels 1..L, which take the multipoles' place
  double* Lx = Mx;
  tm.begin(FMM_PH_P2M, s);
  launch_p2m(t, tb, qt, Mx, s);
  tm.end(FMM_PH_P2M, s);
  tm.begin(FMM_PH_M2M, s);
  for (int l = L; l >= 2; --l) launch_m2m(t, l, tb, Mx, s);
  tm.end(FMM_PH_M2M, s);
  tm.begin(FMM_PH_M2L, s);
  launch_m2l(t, tb, Mx, Lx, prec, s);
  tm.end(FMM_PH_M2L, s);
  tm.begin(FMM_PH_L2L, s);
  for (int l = 2; l <= L; ++l) launch_l2l(t, l, tb, Lx, s);
  tm.end(FMM_PH_L2L, s);
  // after M2L has given back its copy of the multipoles
  for (int k = 0; k < 4; ++k) far[k] = (double*)dalloc(std::max<int64_t>(1, npts) * sizeof(double), s);
  tm.begin(FMM_PH_L2P, s);
  launch_l2p(t, tb, Lx, start, px, py, pz, far[0], far[1], far[2], far[3], s);
  tm.end(FMM_PH_L2P, s);
  dfree(Mx, s);
}

// Near field (P2P) at the points grouped by leaf as [start[b], start[b+1]) of
// (px, py, pz), plus the far field when far[0] is set; results go to index
// perm[.] of the outputs.  leaf_part / npart: partial-sum layout of the split
// leaves for these points.
void near_field_and_store(const Tree& t, const double* qt, int parts, int prec, const int32_t* start,
                          const double* px, const double* py, const double* pz, const int32_t* perm,
                          const int64_t* leaf_part, int64_t npart, double* const far[4], double* pot, double* ex,
                          double* ey, double* ez, hipStream_t s) {
  PhaseTimer& tm = timer();
  const Level& V = t.lev[t.L];
  tm.begin(FMM_PH_P2P, s);
  const unsigned gfin = (unsigned)((V.nbox + 3) / 4);
  if (parts & FMM_PART_NEAR) {
    double4* part = npart > 0 ? (double4*)dalloc(npart * sizeof(double4), s) : nullptr;
    const unsigned grid = (unsigned)(8 * ((t.p2p_nseg + 7) / 8));
    // A block takes its leaf's targets 64 to 256 at a time; where leaves may
    // hold more (cells off the median, separate targets, few levels) and the
    // segments alone leave the chip idle, blocks in y share these passes: the
    // largest leaf held the launch (30,011 targets, 512 leaves off the median
    // 1,750 -> 993 us; blocks without a pass end at once).
    const bool even = start == V.start && t.eta == 1.0;
    const int64_t most = even ? (t.n + V.nbox - 1) / V.nbox : INT64_MAX;  // targets of a leaf
    const int64_t cap = t.p2p_nseg <= 2048 ? 16 : t.p2p_nseg <= 16384 ? 4 : 1;
    const unsigned gy = most <= (prec == FMM_PREC_F32 ? 128 : 256) ? 1 : (unsigned)std::min(cap, (most - 1) / 64 + 1);
    auto go = [&](auto f32, auto w) {
      k_p2p<decltype(f32)::value, decltype(w)::value><<<dim3(grid, gy), 64 * decltype(w)::value, 0, s>>>(
          t.p2p_nseg, t.p2p_seg_leaf, t.p2p_seg_e0, t.p2p_leaf_seg, leaf_part, V.start, V.s_off, V.s_idx, t.px, t.py,
          t.pz, qt, start, px, py, pz, perm, far[0], far[1], far[2], far[3], part, pot, ex, ey, ez, V.geom);
    };
    auto go_w = [&](auto f32) {
      const int w = rules::p2p_waves(t.p2p_nseg, V.s_nnz, decltype(f32)::value);
      if (w == 8)
        go(f32, std::integral_constant<int, 8>{});
      else if (w == 4)
        go(f32, std::integral_constant<int, 4>{});
      else
        go(f32, std::integral_constant<int, 1>{});
    };
    if (prec == FMM_PREC_F32)
      go_w(std::true_type{});
    else
      go_w(std::false_type{});
    HIPCHECK(hipGetLastError());
    if (part) {
      k_p2p_final<1><<<gfin, 256, 0, s>>>(V.nbox, start, t.p2p_leaf_seg, leaf_part, part, perm, far[0], far[1],
                                         far[2], far[3], pot, ex, ey, ez);
      HIPCHECK(hipGetLastError());
      dfree(part, s);
    }
  } else {
    k_p2p_final<0><<<gfin, 256, 0, s>>>(V.nbox, start, nullptr, nullptr, nullptr, perm, far[0], far[1], far[2],
                                       far[3], pot, ex, ey, ez);
    HIPCHECK(hipGetLastError());
  }
  tm.end(FMM_PH_P2P, s);
}

double* gather_charges(const Tree& t, const double* q, hipStream_t s) {
  double* qt = (double*)dalloc(t.n * sizeof(double), s);
  k_gather<<<(unsigned)((t.n + 255) / 256), 256, 0, s>>>(q, t.perm, qt, t.n);
  HIPCHECK(hipGetLastError());
  return qt;
}

}  // namespace

void evaluate(const Tree& t, const double* q, int p, int parts, int prec, double* pot, double* ex, double* ey,
              double* ez, hipStream_t s) {
  double* qt = gather_charges(t, q, s);
  double* far[4] = {nullptr, nullptr, nullptr, nullptr};
  const Level& V = t.lev[t.L];
  if ((parts & FMM_PART_FAR) && t.L >= 1) far_field(t, qt, p, prec, V.start, t.px, t.py, t.pz, t.n, far, s);
  near_field_and_store(t, qt, parts, prec, V.start, t.px, t.py, t.pz, t.perm, t.p2p_leaf_part, t.p2p_npart, far, pot, ex,
                       ey, ez, s);
  for (int k = 0; k < 4; ++k)
    if (far[k]) dfree(far[k], s);
  dfree(qt, s);
}

namespace {
// What an evaluation of the given parts at npts points holds: the charges all
// along; for the far field the expansions with M2L's copy of the multipoles and
// its queue, then the expansions with the far field, then the far field with
// the near field's partial sums.  In one block the expansions' place is not
// used again.
size_t scratch_bytes(const Tree& t, int p, int prec, int parts, int64_t npts, int64_t npart, bool one_block) {
  const size_t qt = (size_t)t.n * 8;
  const size_t part = parts & FMM_PART_NEAR ? (size_t)std::max<int64_t>(0, npart) * 32 : 0;
  if (!(parts & FMM_PART_FAR) || t.L == 0) return qt + part;
  const size_t stride = p <= tl::kMaxP ? (size_t)tl::stride(p) : (size_t)nterms(p);
  const size_t nbox = (size_t)t.nbox_total;
  // the copy, per box: binary32 dense (per-lane kernel, orders up to 14) or
  // tiled (order 15), else binary64 in the quad layout
  size_t copy;
  if (prec != FMM_PREC_F64 && p <= 14) copy = (size_t)lops::dense_stride(p) * 4;
  else if (prec != FMM_PREC_F64 && p <= tl::kMaxP) copy = stride * 4;
  else copy = (size_t)lops::nq(p) * 4 * 8;
  const size_t expn = nbox * stride * 8, far = 4 * (size_t)std::max<int64_t>(1, npts) * 8;
  const size_t m2l = expn + 256 + nbox * copy;
  return qt + (one_block ? std::max(m2l, expn + far + part) : std::max({m2l, expn + far, far + part}));
}
}  // namespace

size_t arena_bytes(const Tree& t, int p, int prec, int parts, bool targets) {
  // at most 12 buffers; each may lose 255 bytes to alignment
  return scratch_bytes(t, p, prec, parts, targets ? t.m : t.n, targets ? t.p2p_ntpart : t.p2p_npart, true) + 12 * 256;
}

size_t eval_scratch_bytes(const Tree& t, int p, int prec) {
  auto one = [&](bool targets) {
    const size_t a = arena_bytes(t, p, prec, FMM_PART_ALL, targets);
    return a <= kOneBlock ? a
                          : scratch_bytes(t, p, prec, FMM_PART_ALL, targets ? t.m : t.n,
                                          targets ? t.p2p_ntpart : t.p2p_npart, false);
  };
  return t.m > 0 ? std::max(one(false), one(true)) : one(false);
}

// phi and E at the tree's separate targets (outputs in the caller's target
// order): the same passes, with L2P and P2P at the targets grouped by leaf
void evaluate_targets(const Tree& t, const double* q, int p, int parts, int prec, double* pot, double* ex, double* ey,
                      double* ez, hipStream_t s) {
  if (t.m == 0) return;
  double* qt = gather_charges(t, q, s);
  double* far[4] = {nullptr, nullptr, nullptr, nullptr};
  if ((parts & FMM_PART_FAR) && t.L >= 1) far_field(t, qt, p, prec, t.tstart, t.tx, t.ty, t.tz, t.m, far, s);
  near_field_and_store(t, qt, parts, prec, t.tstart, t.tx, t.ty, t.tz, t.tperm, t.p2p_leaf_tpart, t.p2p_ntpart, far, pot,
                       ex, ey, ez, s);
  for (int k = 0; k < 4; ++k)
    if (far[k]) dfree(far[k], s);
  dfree(qt, s);
}

}  // namespace fmm
