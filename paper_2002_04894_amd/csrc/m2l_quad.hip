// M2L in binary64 (Algorithm 3, M2L; rotational form of Section 2.1.3), four
// lanes per weak pair, the fixed quarter turns on the matrix cores.
//
// The translation is the sequence of the other M2L kernels:
//   Rz(-beta), J^T, Rz(-alpha), J, z-axis translation, J^T, Rz(alpha), J, Rz(beta),
// with J the fixed quarter turn about x and (alpha, beta) the polar and
// azimuthal angles of d = c_source - c_target, on radius-scaled expansions
// (M~_n = M_n / r_s^n in, the factors (r_s/rho)^n and (r_t/rho)^j / rho, the
// result unscaled by r_t^-n), here all in binary64.
//
// A wave takes 16 pairs of one target box; lane 16 k + q holds phase k of
// pair q (lane_ops.h: per degree two blocks indexed by the order m, the two
// parity classes of J, their even and odd orders in registers of their own).
// Hence:
//   - a J block is a chain of v_mfma_f64_4x4x4f64, one per (k-step, output
//     chunk of 4 rows): the instruction's k index runs over the four phase
//     lanes of a pair, and its output row i lands in phase i of the same pair,
//     so every step's result is the next step's operand in place; the
//     operator values come from LDS (binary64 instructions take no broadcast
//     of one block's operand, so every lane reads its value); the parts that
//     join orders of the wrong parity are zero and left out (360 instead of
//     576 instructions per batch at order 12); J^T has a
//     table of its own up to order 18 and above reads the table of J with
//     the two chunk indices swapped and each 4x4 part transposed;
//   - a z-turn multiplies the (cosine, sine) parts of (d, m), which share a
//     lane and register, by the lane's own e^{i m theta};
//   - the z translation of order m involves only order-m coefficients of
//     all degrees, which share a lane once the even and odd registers have
//     exchanged halves: each lane runs it for its orders on the vector units (binary64 vector and matrix peaks are equal on this part);
//   - the 16 pair results are summed across the lanes by halving exchanges
//     through DPP (fixed order: deterministic) and the batches in binary64.
// What bounds it: binary64 matrix and vector issue (order 12, 2^27 points: 34 and
// 44 % of the cycles); from order 15 on a few values still spill, and above
// it one wave per SIMD hides no latency.  Measured on 2^22 Plummer points (5
// levels, theta 0.6, 194 million pairs), M2L in ms: order 8 38, 10 59, 12 87,
// 13 102, 14 120, 15 154, 16 289, 18 574, 20 833; with whole blocks of J and
// values spilled instead of parked 46, 68, 106, 150, -, -, 375, 703, 1,091, and
// in 16x16 tiles of two degree blocks 178 and 190 at orders 14 and 15.
//
// The same steps with the M2M or L2L core along z make k_xlate_quad (end of
// the file), which runs M2M and L2L up to order 18.
#include <type_traits>

#include "fmm_internal.h"
#include "lane_ops.h"
#include "m2l_queue.h"
#include "tile_layout.h"

namespace fmm {
namespace {

template <int B, int E, class F>
__device__ __forceinline__ void qfor(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    qfor<B + 1, E>(f);
  }
}

// sizes of the halving exchanges over the 16 pairs of a wave
__host__ __device__ constexpr int qlvl(int nt, int s) {
  int v = nt;
  for (int k = 0; k < s; ++k) v = (v + 1) / 2;
  return v;
}

__device__ __forceinline__ double mfma64(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// One block (d, x) of a J application: NR = qreg(d) input registers times NR
// output registers, less the parts without nonzero entries; tl = the lane's slot in a 16-value operand, 4 k + i, or with T
// (J^T from the table of J, whose part (c, g) transposed is part (g, c) of
// J^T) 4 i + k
template <int D, int X>
struct QBlk {
  static constexpr int NR = lops::qreg(D);
  static constexpr int R0 = lops::qbase(D, X);
  static constexpr int U0 = lops::qp_offset(D, X);
  double acc[NR];
  __device__ __forceinline__ QBlk() {
    qfor<0, NR>([&](auto c) __attribute__((always_inline)) { acc[c] = 0.0; });
  }
  template <bool T, int G>
  __device__ __forceinline__ void step(const double* X_, const double* tab, int tl) {
    if constexpr (G < NR) {
      const double xg = X_[R0 + G];
      qfor<0, NR>([&](auto c) __attribute__((always_inline)) {
        constexpr int C = decltype(c)::value;
        if constexpr (lops::qpart(D, X, G, C)) {
          constexpr int u = U0 + (T ? lops::qpart_rank(D, X, C, G) : lops::qpart_rank(D, X, G, C));
          acc[c] = mfma64(tab[16 * u + tl], xg, acc[c]);
        }
      });
    }
  }
  __device__ __forceinline__ void store(double* X_) {
    qfor<0, NR>([&](auto c) __attribute__((always_inline)) { X_[R0 + decltype(c)::value] = acc[c]; });
  }
};

// X <- J X (or J^T X from its own table; T: J^T X from the table of J, tl the
// lane's slot for that case): degree d beside degree P - d, both blocks each,
// in lock-step over the k-steps (independent chains in flight)
template <int P, bool T>
__device__ __forceinline__ void qjapply(double* X, const double* tab, int tl) {
  qfor<0, P / 2 + 1>([&](auto dI) __attribute__((always_inline)) {
    constexpr int d = decltype(dI)::value, d2 = P - d;
    QBlk<d, 0> a0;
    QBlk<d, 1> a1;
    if constexpr (d2 > d) {
      QBlk<d2, 0> b0;
      QBlk<d2, 1> b1;
      qfor<0, lops::qreg(d2)>([&](auto g) __attribute__((always_inline)) {
        constexpr int G = decltype(g)::value;
        a0.template step<T, G>(X, tab, tl);
        a1.template step<T, G>(X, tab, tl);
        b0.template step<T, G>(X, tab, tl);
        b1.template step<T, G>(X, tab, tl);
      });
      b0.store(X);
      b1.store(X);
    } else {
      qfor<0, lops::qreg(d)>([&](auto g) __attribute__((always_inline)) {
        constexpr int G = decltype(g)::value;
        a0.template step<T, G>(X, tab, tl);
        a1.template step<T, G>(X, tab, tl);
      });
    }
    a0.store(X);
    a1.store(X);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// X <- Rz(sign * theta) X with (c1, s1) = (cos theta, sin theta): each member
// turns by e^{i m theta} of its order m; with block 0 holding c_m for even m
// and s_m for odd m, the turn of (b0, b1) is (C b0 - S' b1, S' b0 + C b1) with
// S' = S for even m and -S for odd m.  Per eight orders a lane holds one of the
// even orders (8 b + 2 k), one of the odd (8 b + 2 k + 1) and, in a shared
// register, one of the lowest four.
template <int P>
__device__ __forceinline__ void qrotz(double* X, double c1, double s1, double sign, int k) {
  constexpr int NB = P / 8 + 1;
  const double c2 = c1 * c1 - s1 * s1, s2 = 2.0 * s1 * c1;
  const double c3 = c2 * c1 - s2 * s1, s3 = s2 * c1 + c2 * s1;
  const double c4 = c2 * c2 - s2 * s2, s4 = 2.0 * s2 * c2;
  const double c6 = c4 * c2 - s4 * s2, s6 = s4 * c2 + c4 * s2;
  const double c8 = c4 * c4 - s4 * s4, s8 = 2.0 * s4 * c4;
  double C[NB][3], S[NB][3];  // even, odd, shared
  C[0][0] = k == 0 ? 1.0 : k == 1 ? c2 : k == 2 ? c4 : c6;
  S[0][0] = sign * (k == 0 ? 0.0 : k == 1 ? s2 : k == 2 ? s4 : s6);
  C[0][1] = C[0][0] * c1 - sign * S[0][0] * s1;
  S[0][1] = -(S[0][0] * c1 + sign * C[0][0] * s1);
  C[0][2] = k < 2 ? C[0][0] : k == 2 ? c1 : c3;
  S[0][2] = k < 2 ? S[0][0] : -sign * (k == 2 ? s1 : s3);
#pragma unroll
  for (int b = 1; b < NB; ++b)
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      // the signed sine of an odd order turns the other way
      const double sg = t == 0 ? sign : t == 1 ? -sign : (k < 2 ? sign : -sign);
      C[b][t] = C[b - 1][t] * c8 - sg * S[b - 1][t] * s8;
      S[b][t] = S[b - 1][t] * c8 + sg * C[b - 1][t] * s8;
    }
  qfor<0, P + 1>([&](auto dI) __attribute__((always_inline)) {
    constexpr int d = decltype(dI)::value;
    qfor<0, lops::qreg(d)>([&](auto g) __attribute__((always_inline)) {
      constexpr int G = decltype(g)::value;
      constexpr int t = lops::qpaired(d, G) ? G & 1 : 2;
      constexpr int r0 = lops::qbase(d, 0) + G, r1 = lops::qbase(d, 1) + G;
      const double b0 = X[r0], b1 = X[r1];
      X[r0] = C[G / 2][t] * b0 - S[G / 2][t] * b1;
      X[r1] = S[G / 2][t] * b0 + C[G / 2][t] * b1;
    });
  });
}

// exchanges the two halves of the wave between the even and the odd register
// of every pair: (even, odd orders) <-> (lower, upper four of the eight)
template <int P>
__device__ __forceinline__ void qsort_orders(double* X) {
  qfor<4, P + 1>([&](auto dI) __attribute__((always_inline)) {
    constexpr int d = decltype(dI)::value;
    qfor<0, lops::qreg(d) / 2>([&](auto bI) __attribute__((always_inline)) {
      qfor<0, 2>([&](auto xI) __attribute__((always_inline)) {
        constexpr int r = lops::qbase(d, decltype(xI)::value) + 2 * decltype(bI)::value;
        const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(X[r]), __double2loint(X[r + 1]), false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(X[r]), __double2hiint(X[r + 1]), false, false);
        X[r] = __hiloint2double(h[0], l[0]);
        X[r + 1] = __hiloint2double(h[1], l[1]);
      });
    });
  });
}

// the z-axis translation: the lane's orders m = 4 g + qshared(k), both blocks
// (the registers sorted by order meanwhile), with
// the core A[m][d][n] of its own order (Az, orders above P zero).  Input
// degree n is first multiplied by in_base^n and output degree d by out_mult
// out_base^d; with EXP also by 2^(in_exp n) and 2^(out_exp d) (ldexp: exact,
// and saturating only where the scaled value itself leaves the range)
template <int P, bool EXP = false>
__device__ __forceinline__ void qztrans(double* X, const double* __restrict__ Az, int k, double in_base,
                                        double out_base, double out_mult, int in_exp = 0, int out_exp = 0) {
  constexpr int P1 = P + 1;
  {
    double w = 1.0;
    qfor<0, P + 1>([&](auto dI) __attribute__((always_inline)) {
      constexpr int d = decltype(dI)::value;
      qfor<0, 2 * lops::qreg(d)>([&](auto r) __attribute__((always_inline)) {
        if constexpr (EXP)
          X[lops::qbase(d, 0) + decltype(r)::value] = ldexp(X[lops::qbase(d, 0) + decltype(r)::value] * w, in_exp * d);
        else
          X[lops::qbase(d, 0) + decltype(r)::value] *= w;
      });
      w *= in_base;
    });
  }
  qsort_orders<P>(X);
  const int ks = lops::qshared(k);
  qfor<0, P / 4 + 1>([&](auto gI) __attribute__((always_inline)) {
    constexpr int G = decltype(gI)::value;
    constexpr int N0 = 4 * G;  // lowest degree holding register G
    // the lane's order, orders above P reading the zero slot P + 1
    const double* Am = Az + (4 * G + ks <= P ? 4 * G + ks : P + 1) * P1 * P1;
    double y0[P1 - N0], y1[P1 - N0];
    qfor<0, P1 - N0>([&](auto r) __attribute__((always_inline)) { y0[r] = y1[r] = 0.0; });
    // input degree by input degree: only one column of the core is loaded
    // at a time (all of them at once would not fit the registers)
    qfor<N0, P1>([&](auto nI) __attribute__((always_inline)) {
      constexpr int n = decltype(nI)::value;
      const double x0 = X[lops::qbase(n, 0) + G], x1 = X[lops::qbase(n, 1) + G];
      qfor<N0, P1>([&](auto dI) __attribute__((always_inline)) {
        constexpr int d = decltype(dI)::value;
        const double a = Am[d * P1 + n];
        y0[d - N0] += a * x0;
        y1[d - N0] += a * x1;
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    qfor<N0, P1>([&](auto dI) __attribute__((always_inline)) {
      constexpr int d = decltype(dI)::value;
      X[lops::qbase(d, 0) + G] = y0[d - N0];
      X[lops::qbase(d, 1) + G] = y1[d - N0];
    });
  });
  qsort_orders<P>(X);
  {
    double w = out_mult;
    qfor<0, P + 1>([&](auto dI) __attribute__((always_inline)) {
      constexpr int d = decltype(dI)::value;
      qfor<0, 2 * lops::qreg(d)>([&](auto r) __attribute__((always_inline)) {
        if constexpr (EXP)
          X[lops::qbase(d, 0) + decltype(r)::value] = ldexp(X[lops::qbase(d, 0) + decltype(r)::value] * w, out_exp * d);
        else
          X[lops::qbase(d, 0) + decltype(r)::value] *= w;
      });
      w *= out_base;
    });
  }
}

__device__ __forceinline__ int qlevel_of(const LevelView& lv, int64_t gid) {
  int l = 0;
  while (l < lv.L && gid >= lv.gofs[l + 1]) ++l;
  return l;
}

// Waves per SIMD: 2 up to order 15, 1 above.  One block per CU (512 threads
// for two waves per SIMD, 256 for one), so that the tables (J, J^T up to order
// 18, the z core) are staged into LDS once per CU, and beside them the values
// that a lane parks while the translation runs: the angles, the distance
// factors, the sums over the batches.
template <int P>
struct QuadCfg {
  static constexpr int kThreads = lops::qthreads(P);
  static constexpr int kWaves = kThreads / 256;
  static constexpr int kJ = 16 * lops::qp_count(P);  // doubles of the J table
  static constexpr int kLds = lops::qp_doubles(P);
  static constexpr int kSums = lops::qsums(P);
  static_assert(kLds * 8 + lops::qpark_bytes(P) <= 160 * 1024, "tables and parked values must fit in LDS");
  static_assert(kSums == qlvl(lops::nq(P), 4) && lops::qp_count(P) <= lops::qj_count(P), "");
};

// One step of the translation, kept apart from its neighbours by the
// scheduler (bounds the registers in flight)
#define FMM_QSTEP(x) \
  x;                 \
  __builtin_amdgcn_sched_barrier(0)

// A halving exchange over lanes at distance D (8, 4, 2 or 1: within a row of
// 16 lanes) of a wave whose lanes hold NS values src: lanes with that lane bit
// clear keep the lower ND values and add their partner's, the others the
// upper ones (zero-padded).  The partner's value is a DPP read (row_ror:8,
// quad_perm [2,3,0,1] or [1,0,3,2]; distance 4 as two shifts, row_shl:4 and
// row_shr:4), vector work instead of LDS permutes, which the operand reads
// already load.
template <int CTRL>
__device__ __forceinline__ double qdpp(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true));
}
template <int NS, int ND, int D>
__device__ __forceinline__ void qhalve(const double* src, double* dst, int lane) {
  const bool up = (lane & D) != 0;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const double lo = src[i];
    const double hi = ND + i < NS ? src[ND + i] : 0.0;
    if constexpr (D == 4) {
      const double t0 = lo + qdpp<0x104>(lo), t1 = hi + qdpp<0x114>(hi);
      dst[i] = up ? t1 : t0;
    } else {
      constexpr int C = D == 8 ? 0x128 : D == 2 ? 0x4E : 0xB1;
      const double send = up ? lo : hi, keep = up ? hi : lo;
      dst[i] = keep + qdpp<C>(send);
    }
    if ((i & 7) == 7) __builtin_amdgcn_sched_barrier(0);
  }
}

// The tables into LDS, 16 bytes per load (NL is even: (p + 2) (p + 1)^2 and
// whole parts), eight loads in flight per thread.
template <int NL, int NTH>
__device__ __forceinline__ void qstage(const double* __restrict__ src, double* dst) {
  static_assert(NL % 2 == 0, "");
  const double2* s = (const double2*)src;
  double2* d = (double2*)dst;
#pragma unroll 8
  for (int i = threadIdx.x; i < NL / 2; i += NTH) d[i] = s[i];
}

// Storage position of the coefficient in (register, phase) = (t / 4, t % 4) and
// its degree times 65536; -1 for a zero slot.  All degrees at once: the loop
// unrolls into a few comparisons.
template <int P>
__device__ __forceinline__ int qslot(int t, const int* __restrict__ pos) {
  const int R = t >> 2, ph = t & 3;
  int w = -1;
  qfor<0, P + 1>([&](auto dI) __attribute__((always_inline)) {
    constexpr int d = decltype(dI)::value;
    if (R >= lops::qbase(d, 0) && R < lops::qbase(d + 1, 0)) {
      const int x = R - lops::qbase(d, 0) >= lops::qreg(d) ? 1 : 0;
      const int g = R - lops::qbase(d, 0) - x * lops::qreg(d);
      const int mi = lops::qmember(d, x, lops::qorder(d, g, ph));
      if (mi >= 0) w = pos[d * d + mi] | (d << 16);
    }
  });
  return w;
}

// SHARE, RUNS: how the targets are dealt out (m2l_queue.h); template arguments,
// as a scalar more in the loop's registers spills at the highest orders
template <int P, bool SHARE, bool RUNS>
__global__ __launch_bounds__(QuadCfg<P>::kThreads)
__attribute__((amdgpu_waves_per_eu(QuadCfg<P>::kWaves, QuadCfg<P>::kWaves))) void
k_m2l_quad(LevelView lv, const double* __restrict__ qtab, const int* __restrict__ pos, int S,
           const double* __restrict__ Mq, double* __restrict__ Lx, int64_t ntarget, const int32_t* __restrict__ order,
           int* __restrict__ queue, const int32_t* __restrict__ nlong) {
  if (SHARE && nlong && (int)blockIdx.x >= *nlong) return;  // not one of the long lists
  constexpr int NQ = lops::nq(P);
  constexpr int NJ = QuadCfg<P>::kJ;
  constexpr int NF = QuadCfg<P>::kSums;  // values a lane holds after the exchanges
  constexpr int NL = QuadCfg<P>::kLds;
  constexpr int NTH = QuadCfg<P>::kThreads;
  __shared__ __align__(16) double tabs[NL];
  __shared__ double park[(6 + NF) * NTH];
  __shared__ int slot[NQ * 4];
  qstage<NL, NTH>(qtab, tabs);
  for (int t = threadIdx.x; t < NQ * 4; t += blockDim.x) slot[t] = qslot<P>(t, pos);
  __syncthreads();
  constexpr bool HJT = lops::qp_has_jt(P);
  const double* Az = tabs + (HJT ? 2 : 1) * NJ;
  const int lane = threadIdx.x & 63;
  const int k = lane >> 4, q = lane & 15;
  const int tl = 4 * k + (lane & 3);   // this lane's value in a 4x4 part of J
  const int tlt = 4 * (lane & 3) + k;  // and of J^T
  m2lq::Cursor<RUNS> cur;
  const int wave = SHARE ? m2lq::uniform((int)(threadIdx.x >> 6)) : 0;
  for (;;) {
    const int64_t kq = SHARE ? (int64_t)blockIdx.x : cur.next(queue, ntarget, lane);
    if (kq >= ntarget) break;
    // the target's data are the same in all lanes: kept in scalar registers
    const int64_t gid = lv.gofs[1] + m2lq::uniform(order[kq]);
    const int l = qlevel_of(lv, gid);
    const int64_t bi = gid - lv.gofs[l];
    const double* geo = lv.geom[l];
    const double cix = m2lq::uniform(geo[bi * 10 + 6]), ciy = m2lq::uniform(geo[bi * 10 + 7]);
    const double ciz = m2lq::uniform(geo[bi * 10 + 8]), rt_ = m2lq::uniform(geo[bi * 10 + 9]);
    const double rt = rt_ > 0.0 ? rt_ : 1.0;
    const int32_t* wrow = lv.w_idx[l] + m2lq::uniform(lv.w_off[l][bi]);
    const int ne = (int)m2lq::uniform(lv.w_off[l][bi + 1] - lv.w_off[l][bi]);
    const double* Mlev = Mq + (size_t)lv.gofs[l] * NQ * 4;
    m2lq::Kept<double, NF, true> acc(park + 6 * NTH + threadIdx.x, NTH);
    m2lq::Kept<double, 6, true> geom(park + threadIdx.x, NTH);  // ca, sa, cb, sb, out_base, out_mult
#pragma unroll
    for (int i = 0; i < NF; ++i) acc.put(i, 0.0);

    // the next batch's source indexes are loaded while this batch runs
    const int b0 = 16 * wave, bs = 16 * (SHARE ? NTH / 64 : 1);
    int32_t jn = ne > 0 ? wrow[b0 + q < ne ? b0 + q : 0] : 0;
    for (int eb = b0; eb < ne; eb += bs) {
      const int e = eb + q;
      const bool valid = e < ne;
      const int64_t j = jn;
      jn = wrow[e + bs < ne ? e + bs : 0];
      const double dx = geo[j * 10 + 6] - cix, dy = geo[j * 10 + 7] - ciy, dz = geo[j * 10 + 8] - ciz;
      const double rs = geo[j * 10 + 9] > 0.0 ? geo[j * 10 + 9] : 1.0;
      const double rxy2 = dx * dx + dy * dy;
      const double irho = m2lq::rsqrt0(rxy2 + dz * dz), irxy = m2lq::rsqrt0(rxy2);
      const double ca = dz * irho, sa = rxy2 * irxy * irho;
      const double cb = rxy2 > 0.0 ? dx * irxy : 1.0, sb = dy * irxy;
      // a pair past the end of the list translates the first source with zero factors
      const double in_base = valid ? rs * irho : 0.0;
      geom.put(0, ca);
      geom.put(1, sa);
      geom.put(2, cb);
      geom.put(3, sb);
      geom.put(4, valid ? rt * irho : 0.0);
      geom.put(5, valid ? irho : 0.0);

      double X[NQ];
      const double* src = Mlev + (size_t)j * NQ * 4 + k;
#pragma unroll
      for (int r = 0; r < NQ; ++r) X[r] = src[4 * r];

      FMM_QSTEP(qrotz<P>(X, cb, sb, -1.0, k));
      FMM_QSTEP((qjapply<P, !HJT>(X, HJT ? tabs + NJ : tabs, HJT ? tl : tlt)));
      FMM_QSTEP(qrotz<P>(X, geom.get(0), geom.get(1), -1.0, k));
      FMM_QSTEP((qjapply<P, false>(X, tabs, tl)));
      FMM_QSTEP(qztrans<P>(X, Az, k, in_base, geom.get(4), geom.get(5)));
      FMM_QSTEP((qjapply<P, !HJT>(X, HJT ? tabs + NJ : tabs, HJT ? tl : tlt)));
      FMM_QSTEP(qrotz<P>(X, geom.get(0), geom.get(1), 1.0, k));
      FMM_QSTEP((qjapply<P, false>(X, tabs, tl)));
      FMM_QSTEP(qrotz<P>(X, geom.get(2), geom.get(3), 1.0, k));

      // sum over the 16 pairs (lane bits 0..3): four halving exchanges
      double h1[qlvl(NQ, 1)], h2[qlvl(NQ, 2)], h3[qlvl(NQ, 3)], h4[qlvl(NQ, 4)];
      qhalve<NQ, qlvl(NQ, 1), 8>(X, h1, lane);
      qhalve<qlvl(NQ, 1), qlvl(NQ, 2), 4>(h1, h2, lane);
      qhalve<qlvl(NQ, 2), qlvl(NQ, 3), 2>(h2, h3, lane);
      qhalve<qlvl(NQ, 3), qlvl(NQ, 4), 1>(h3, h4, lane);
#pragma unroll
      for (int i = 0; i < NF; ++i) acc.put(i, acc.get(i) + h4[i]);
    }
    if constexpr (SHARE) {  // the waves' sums, in wave order
      __syncthreads();
      if (threadIdx.x >= 64) return;
      for (int w = 64; w < NTH; w += 64)
#pragma unroll
        for (int i = 0; i < NF; ++i) acc.put(i, acc.get(i) + park[(6 + i) * NTH + w + lane]);
    }
    // lane's values: registers base + i of phase k, where each exchange
    // added the kept half's offset; entries past a half's end are padding
    int base = 0, len = NQ;
#pragma unroll
    for (int sidx = 1; sidx <= 4; ++sidx) {
      const int half = qlvl(NQ, sidx);
      const int dist = 16 >> sidx;
      if (lane & dist) {
        base += half;
        len = len - half > 0 ? len - half : 0;
      } else {
        len = len < half ? len : half;
      }
    }
    double* dst = Lx + (size_t)gid * S;
    const double irt = 1.0 / rt;
    qfor<0, NF>([&](auto iI) __attribute__((always_inline)) {
      constexpr int i = decltype(iI)::value;
      if (i < len) {
        const int w = slot[4 * (base + i) + k];
        if (w >= 0) {
          double v = acc.get(i);
          for (int t = w >> 16; t > 0; --t) v *= irt;
          dst[w & 0xffff] = v;
        }
      }
    });
    if constexpr (SHARE) return;
  }
}

// The multipoles of levels 1..L in the quad layout, scaled by r^-n (r the box
// radius, 1 for a box of zero extent): per box NQ registers x 4 phases.
template <int P>
__global__ void k_quad_copy(LevelView lv, int S, const int* __restrict__ pos, const double* __restrict__ Mx,
                            double* __restrict__ Mq, int64_t nbox_total) {
  constexpr int NQ = lops::nq(P);
  const int64_t gid = 1 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (gid >= nbox_total) return;
  int l = 1;
  while (l < lv.L && gid >= lv.gofs[l + 1]) ++l;
  const double r = lv.geom[l][(gid - lv.gofs[l]) * 10 + 9];
  const double is = r > 0.0 ? 1.0 / r : 1.0;
  for (int t = threadIdx.x & 63; t < 4 * NQ; t += 64) {
    const int w = qslot<P>(t, pos);
    double v = 0.0;
    if (w >= 0) {
      v = Mx[(size_t)gid * S + (w & 0xffff)];
      for (int u = w >> 16; u > 0; --u) v *= is;
    }
    Mq[(size_t)gid * NQ * 4 + t] = v;
  }
}

__global__ void k_start_queue_q(int* queue, const int32_t* first) {
  if (threadIdx.x < m2lq::kXcds) queue[threadIdx.x] = threadIdx.x == 0 && first ? *first : 0;
}

template <int P>
void launch_one_quad(const Tree& t, const Tables& tb, const double* Mx, double* Lx, hipStream_t s) {
  const int64_t ntarget = t.nbox_total - 1;
  if (ntarget <= 0) return;
  constexpr int NQ = lops::nq(P);
  double* Mq = (double*)dalloc((size_t)t.nbox_total * NQ * 4 * sizeof(double), s);
  k_quad_copy<P><<<(unsigned)((ntarget + 3) / 4), 256, 0, s>>>(t.view(), tb.stride, tb.pos, Mx, Mq, t.nbox_total);
  HIPCHECK(hipGetLastError());
  const int32_t* nlong = ntarget > m2lq::kShareQuad && ntarget <= m2lq::kLongQuad ? t.m2l_order + ntarget : nullptr;
  if (ntarget <= m2lq::kLongQuad) {
    // all targets, or the long lists: at most kM2LWaves of them can be longer
    // than their share
    const unsigned blocks = (unsigned)(nlong && ntarget > kM2LWaves ? kM2LWaves : ntarget);
    k_m2l_quad<P, true, false><<<blocks, QuadCfg<P>::kThreads, 0, s>>>(t.view(), tb.quad, tb.pos, tb.stride, Mq, Lx,
                                                                        ntarget, t.m2l_order, nullptr, nlong);
    HIPCHECK(hipGetLastError());
  }
  if (ntarget > m2lq::kShareQuad) {
    static const int grid_max = [] {
      int dev = 0, ncu = 0;
      HIPCHECK(hipGetDevice(&dev));
      HIPCHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
      return ncu;  // one block per CU, by its LDS and registers
    }();
    const int64_t need = (ntarget + QuadCfg<P>::kThreads / 64 - 1) / (QuadCfg<P>::kThreads / 64);
    const unsigned grid = (unsigned)(need < grid_max ? need : grid_max);
    int* queue = (int*)dalloc(m2lq::kXcds * sizeof(int), s);
    k_start_queue_q<<<1, 64, 0, s>>>(queue, nlong);
    HIPCHECK(hipGetLastError());
    if (ntarget >= kM2LSiblingsMin)
      k_m2l_quad<P, false, true><<<grid, QuadCfg<P>::kThreads, 0, s>>>(t.view(), tb.quad, tb.pos, tb.stride, Mq, Lx,
                                                                       ntarget, t.m2l_order, queue, nullptr);
    else
      k_m2l_quad<P, false, false><<<grid, QuadCfg<P>::kThreads, 0, s>>>(t.view(), tb.quad, tb.pos, tb.stride, Mq, Lx,
                                                                        ntarget, t.m2l_order, queue, nullptr);
    HIPCHECK(hipGetLastError());
    dfree(queue, s);
  }
  dfree(Mq, s);
}

// ---- M2M and L2L, four lanes per translation (Algorithm 1 M2M, Algorithm 3
// L2L; orders up to kQuadXlateMaxP) ----
// The rotations and quarter turns of the M2L kernel with the M2M or L2L core
// along z; the distance powers are applied apart (M2M: input degree n times
// rho^-n, output degree d times rho^d; L2L the reverse), in binary64 without
// radius scaling, each power split into one of mu in [1, 2) and an exact
// power-of-two scaling.  A wave takes 16 children of level l, the children of two
// parents: M2M sums each parent's eight translated children by three halving
// exchanges and writes the parent (and zeroes its storage's padding slots);
// L2L adds the parent's translated expansion into each child.  The vector is
// child centre - parent centre for both, as in the generic translation, and
// a pair at distance zero is the identity (its input is added back).
template <int P, bool L2L>
__global__ __launch_bounds__(QuadCfg<P>::kThreads)
__attribute__((amdgpu_waves_per_eu(QuadCfg<P>::kWaves, QuadCfg<P>::kWaves))) void
k_xlate_quad(LevelView lv, int l, const double* __restrict__ qtab, const int* __restrict__ pos,
             const int* __restrict__ ipos, int S, double* __restrict__ E, int64_t ngroup) {
  constexpr int NQ = lops::nq(P);
  constexpr int NJ = QuadCfg<P>::kJ;
  constexpr int NL = QuadCfg<P>::kLds;
  constexpr int NF = qlvl(NQ, 3);  // values a lane holds after the M2M exchanges
  static_assert(lops::qp_has_jt(P), "orders whose table holds J^T");
  __shared__ __align__(16) double tabs[NL];
  __shared__ int spos[NQ * 4];  // storage position of (register, phase); -1: zero slot
  qstage<NL, QuadCfg<P>::kThreads>(qtab, tabs);
  for (int t = threadIdx.x; t < NQ * 4; t += blockDim.x) {
    const int w = qslot<P>(t, pos);
    spos[t] = w >= 0 ? w & 0xffff : -1;
  }
  __syncthreads();
  const double* Az = tabs + 2 * NJ;
  const int lane = threadIdx.x & 63;
  const int k = lane >> 4, q = lane & 15;
  const int tl = 4 * k + (lane & 3);
  const double* gch = lv.geom[l];
  const double* gpa = lv.geom[l - 1];
  // few groups are spread over blocks first: a wave by itself on its SIMD
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t cg = (int64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x; cg < ngroup; cg += nw) {
    const int64_t ch = 16 * cg + q, par = ch >> 3;
    const double dx = gch[ch * 10 + 6] - gpa[par * 10 + 6];
    const double dy = gch[ch * 10 + 7] - gpa[par * 10 + 7];
    const double dz = gch[ch * 10 + 8] - gpa[par * 10 + 8];
    const double rxy2 = dx * dx + dy * dy;
    const double rho = sqrt(rxy2 + dz * dz), rxy = sqrt(rxy2);
    const bool zero = !(rho > 0.0);
    const double ca = zero ? 1.0 : dz / rho, sa = zero ? 0.0 : rxy / rho;
    const double cb = rxy > 0.0 ? dx / rxy : 1.0, sb = rxy > 0.0 ? dy / rxy : 0.0;
    // rho = 2^e mu with mu in [1, 2): the powers of mu stay in range and
    // those of 2^e are exact ldexp scalings, so no partial product leaves the
    // binary64 range unless the scaled coefficient does.  A pair at distance
    // zero translates to zero here; its identity is added below.
    const int e = zero ? 0 : ilogb(rho);
    const double mu = zero ? 0.0 : ldexp(rho, -e);
    const double in_base = zero ? 0.0 : (L2L ? mu : 1.0 / mu);
    const double out_base = zero ? 0.0 : (L2L ? 1.0 / mu : mu);
    const double out_mult = zero ? 0.0 : 1.0;
    const int in_exp = L2L ? e : -e, out_exp = -in_exp;
    const double* src = E + (size_t)(L2L ? lv.gofs[l - 1] + par : lv.gofs[l] + ch) * S;

    double X[NQ];
    qfor<0, NQ>([&](auto rI) __attribute__((always_inline)) {
      const int sp = spos[4 * decltype(rI)::value + k];
      X[decltype(rI)::value] = sp >= 0 ? src[sp] : 0.0;
    });
    FMM_QSTEP(qrotz<P>(X, cb, sb, -1.0, k));
    FMM_QSTEP((qjapply<P, false>(X, tabs + NJ, tl)));
    FMM_QSTEP(qrotz<P>(X, ca, sa, -1.0, k));
    FMM_QSTEP((qjapply<P, false>(X, tabs, tl)));
    FMM_QSTEP((qztrans<P, true>(X, Az, k, in_base, out_base, out_mult, in_exp, out_exp)));
    FMM_QSTEP((qjapply<P, false>(X, tabs + NJ, tl)));
    FMM_QSTEP(qrotz<P>(X, ca, sa, 1.0, k));
    FMM_QSTEP((qjapply<P, false>(X, tabs, tl)));
    FMM_QSTEP(qrotz<P>(X, cb, sb, 1.0, k));
    if (__ballot(zero)) {
      qfor<0, NQ>([&](auto rI) __attribute__((always_inline)) {
        const int sp = spos[4 * decltype(rI)::value + k];
        if (zero && sp >= 0) X[decltype(rI)::value] += src[sp];
      });
    }

    if constexpr (L2L) {
      double* dst = E + (size_t)(lv.gofs[l] + ch) * S;
      qfor<0, NQ>([&](auto rI) __attribute__((always_inline)) {
        const int sp = spos[4 * decltype(rI)::value + k];
        if (sp >= 0) dst[sp] += X[decltype(rI)::value];
      });
    } else {
      // sum over the eight children of each parent (lane bits 0..2)
      double h1[qlvl(NQ, 1)], h2[qlvl(NQ, 2)], h3[qlvl(NQ, 3)];
      qhalve<NQ, qlvl(NQ, 1), 4>(X, h1, lane);
      qhalve<qlvl(NQ, 1), qlvl(NQ, 2), 2>(h1, h2, lane);
      qhalve<qlvl(NQ, 2), qlvl(NQ, 3), 1>(h2, h3, lane);
      // lane's values: registers base + i of phase k of parent 2 cg + (q >> 3)
      int base = 0, len = NQ;
#pragma unroll
      for (int sidx = 1; sidx <= 3; ++sidx) {
        const int half = qlvl(NQ, sidx);
        if (lane & (8 >> sidx)) {
          base += half;
          len = len - half > 0 ? len - half : 0;
        } else {
          len = len < half ? len : half;
        }
      }
      double* dst = E + (size_t)(lv.gofs[l - 1] + 2 * cg + (q >> 3)) * S;
      qfor<0, NF>([&](auto iI) __attribute__((always_inline)) {
        constexpr int i = decltype(iI)::value;
        if (i < len) {
          const int sp = spos[4 * (base + i) + k];
          if (sp >= 0) dst[sp] = h3[i];
        }
      });
      double* pdst = E + (size_t)(lv.gofs[l - 1] + 2 * cg) * S;
      for (int t = lane; t < 2 * S; t += 64)
        if (ipos[t % S] < 0) pdst[t] = 0.0;
    }
  }
}

template <int P, bool L2L>
void launch_one_xlate(const Tree& t, int l, const Tables& tb, double* E, hipStream_t s) {
  const int64_t ngroup = t.lev[l].nbox / 16;
  if (ngroup <= 0) return;
  static const int grid_max = [] {
    int dev = 0, ncu = 0, per = 0;
    HIPCHECK(hipGetDevice(&dev));
    HIPCHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    HIPCHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_xlate_quad<P, L2L>, QuadCfg<P>::kThreads, 0));
    return ncu * (per > 0 ? per : 1);
  }();
  const unsigned grid = (unsigned)(ngroup < grid_max ? ngroup : grid_max);
  k_xlate_quad<P, L2L><<<grid, QuadCfg<P>::kThreads, 0, s>>>(t.view(), l, L2L ? tb.quad_l2l : tb.quad_m2m, tb.pos,
                                                              tb.ipos, tb.stride, E, ngroup);
  HIPCHECK(hipGetLastError());
}

// The build compiles this file once for each PART of the orders, PART, PART +
// kQuadParts, ..., as all of them in one unit would take most of its time.
constexpr int kQuadParts = 4;
template <int P>
bool m2l_from(const Tree& t, const Tables& tb, const double* Mx, double* Lx, hipStream_t s) {
  if constexpr (P > kMaxOrder) {
    return false;
  } else {
    if (tb.p != P) return m2l_from<P + kQuadParts>(t, tb, Mx, Lx, s);
    launch_one_quad<P>(t, tb, Mx, Lx, s);
    return true;
  }
}
template <int P, bool L2L>
bool xlate_from(const Tree& t, int l, const Tables& tb, double* E, hipStream_t s) {
  if constexpr (P > kQuadXlateMaxP) {
    return false;
  } else {
    if (tb.p != P) return xlate_from<P + kQuadParts, L2L>(t, l, tb, E, s);
    launch_one_xlate<P, L2L>(t, l, tb, E, s);
    return true;
  }
}

}  // namespace

// the part's kernel of order tb.p; false if it has none
template <int PART>
bool quad_m2l(const Tree& t, const Tables& tb, const double* Mx, double* Lx, hipStream_t s) {
  return m2l_from<PART>(t, tb, Mx, Lx, s);
}
template <int PART, bool L2L>
bool quad_xlate(const Tree& t, int l, const Tables& tb, double* E, hipStream_t s) {
  return xlate_from<PART, L2L>(t, l, tb, E, s);
}
#define FMM_QUAD_PART(EXTERN, PART)                                                                     \
  EXTERN template bool quad_m2l<PART>(const Tree&, const Tables&, const double*, double*, hipStream_t); \
  EXTERN template bool quad_xlate<PART, false>(const Tree&, int, const Tables&, double*, hipStream_t);  \
  EXTERN template bool quad_xlate<PART, true>(const Tree&, int, const Tables&, double*, hipStream_t);
#ifdef FMM_PART
FMM_QUAD_PART(, FMM_PART)
#endif

#if !defined(FMM_PART) || FMM_PART == 0
static_assert(kQuadParts == 4, "the parts named here");
#ifdef FMM_PART
FMM_QUAD_PART(extern, 1)
FMM_QUAD_PART(extern, 2)
FMM_QUAD_PART(extern, 3)
#endif

// binary64 M2L with this kernel, at every order
bool launch_m2l_quad64(const Tree& t, const Tables& tb, const double* Mx, double* Lx, hipStream_t s) {
  return quad_m2l<0>(t, tb, Mx, Lx, s) || quad_m2l<1>(t, tb, Mx, Lx, s) || quad_m2l<2>(t, tb, Mx, Lx, s) ||
         quad_m2l<3>(t, tb, Mx, Lx, s);
}

namespace {
template <bool L2L>
bool launch_xlate(const Tree& t, int l, const Tables& tb, double* E, hipStream_t s) {
  return quad_xlate<0, L2L>(t, l, tb, E, s) || quad_xlate<1, L2L>(t, l, tb, E, s) ||
         quad_xlate<2, L2L>(t, l, tb, E, s) || quad_xlate<3, L2L>(t, l, tb, E, s);
}
}  // namespace

// M2M from level l into level l - 1, or L2L from level l - 1 into level l,
// four lanes per translation: orders up to kQuadXlateMaxP with the tables
// made; false for the others (the generic translation then runs)
bool launch_m2m_quad64(const Tree& t, int l, const Tables& tb, double* Mx, hipStream_t s) {
  return tb.quad_m2m != nullptr && t.lev[l].nbox % 16 == 0 && launch_xlate<false>(t, l, tb, Mx, s);
}
bool launch_l2l_quad64(const Tree& t, int l, const Tables& tb, double* Lx, hipStream_t s) {
  return tb.quad_l2l != nullptr && t.lev[l].nbox % 16 == 0 && launch_xlate<true>(t, l, tb, Lx, s);
}
#endif

}  // namespace fmm
