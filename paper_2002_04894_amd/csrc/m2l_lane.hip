// M2L for the mixed-precision mode (Algorithm 3, M2L; rotational form of
// Section 2.1.3), one weak pair per lane, at orders p <= 14: binary32 on
// radius-scaled expansions, the fixed operators on the matrix cores.
//
// Every lane of a wave takes one pair of the same target box, 64 pairs at a
// time, and holds its pair's whole expansion in registers in the standard
// order (c_{n,0}, c_{n,1}, s_{n,1}, ..., per degree n).  The translation is
// the same sequence as in the binary64 kernels:
//   Rz(-beta), J^T, Rz(-alpha), J, z-axis translation, J^T, Rz(alpha), J, Rz(beta),
// with J the fixed quarter turn about x (block-diagonal in two parity classes
// per degree) and (alpha, beta) the polar and azimuthal angles of
// d = c_source - c_target.  J, J^T and the z-translation core are the same
// for every pair, so each of their blocks acts on all 64 lanes at once as a
// chain of 4x4x1 matrix instructions (16 blocks of 4 lanes): one instruction
// multiplies four operator rows by one coefficient of every lane, and its
// four results land in that lane's registers -- lane = pair, register = row,
// no data moves between lanes.  The operator values of 16 instructions share
// one register (one block's values broadcast to all blocks, lane_ops.h),
// read from a table in LDS.  Half the entries of a class block of J vanish (the
// turn carries reflections in y into reflections in z), so a class runs as two
// sub-blocks by the parity of the order: 1,500 instructions per batch at p =
// 12, where whole blocks take 2,140.  Only rows of a block are padded to a
// multiple of 4.  The z-turns and the radius powers run on
// the vector units.  The 64 pair results are summed across the lanes by
// halving exchanges (a fixed order: deterministic) and the batch sums are
// added in binary64.  The expansions are scaled as for the binary32 tile
// kernel: M~_n = M_n / r_s^n on the way in, so the factors (r_s/rho)^n and
// (r_t/rho)^j / rho stay below one, and the result is unscaled by r_t^-n
// into binary64.
#include <tuple>
#include <type_traits>

#include "fmm_internal.h"
#include "lane_ops.h"
#include "m2l_queue.h"
#include "tile_layout.h"

namespace fmm {
namespace {

__host__ __device__ constexpr int deg_of(int k) {
  int n = 0;
  while ((n + 1) * (n + 1) <= k) ++n;
  return n;
}
// index of c_{n,m} (t = 0) or s_{n,m} (t = 1) in the standard order
__host__ __device__ constexpr int cidx(int n, int m, int t) { return n * n + (m == 0 ? 0 : 2 * m - 1 + t); }
// sizes of the halving exchanges: level 0 holds all NT values, each of the
// six levels keeps the lane's half (rounded up)
__host__ __device__ constexpr int lvl(int nt, int s) {
  int v = nt;
  for (int k = 0; k < s; ++k) v = (v + 1) / 2;
  return v;
}

typedef float f4 __attribute__((ext_vector_type(4)));

// D + A_ab * b on the 16-block 4x4x1 instruction, the A operand of block AB
// broadcast to all blocks: lane 4q + j receives rows i = 0..3 of
// A_AB[i] * b(lane)
template <int AB>
__device__ __forceinline__ f4 mfma_bc(float a, float b, f4 d) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, d, 4, AB, 0);
}

// f(integral_constant<int, I>) for I = B .. E-1, as straight-line code
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Blocks on the matrix cores.  A block B of kCols inputs x_k = X[in(k)] and
// kRows results computes D_c += Op[4c .. 4c+3][k] x_k, then sets X[out(r)] =
// row r.  The blocks of one call run in lock-step over k, so that their
// accumulator chains are independent instructions in flight; all inputs are
// read before any result is stored, and a block without columns is absent.
// The instructions are numbered in the order of issue (u(k) the first one of
// column k, or of the one ahead of it that j_lead keeps), sixteen to an
// operand register; Ops, carried from block to block,
// holds the current register and the next one, loaded sixteen instructions
// ahead so that its LDS latency is covered.
struct Ops {
  float cur, next;
  const float* tab;
  int lane;
  __device__ __forceinline__ Ops(const float* t, int l) : cur(0.f), next(t[l]), tab(t), lane(l) {}
  // before instruction U is issued, with PREV the one issued before it (-1:
  // none) and E the last of the sequence
  template <int U, int PREV, int E>
  __device__ __forceinline__ void at() {
    constexpr int G = U / 16, GP = PREV < 0 ? -1 : PREV / 16;
    if constexpr (G != GP) {
      cur = G == GP + 1 ? next : tab[G * 64 + lane];
      if constexpr (G < E / 16) next = tab[(G + 1) * 64 + lane];
    }
  }
};

template <class B>
struct Acc {
  static constexpr int kNC = B::kRows > 0 ? lops::chunks(B::kRows) : 1;
  f4 D[kNC];
  __device__ __forceinline__ Acc() {
    static_for<0, kNC>([&](auto c) __attribute__((always_inline)) { D[c] = f4{0.f, 0.f, 0.f, 0.f}; });
  }
  template <int K>
  __device__ __forceinline__ void step(const float* X, Ops& ops) {
    if constexpr (K < B::kCols) {
      constexpr int U = B::u(K) + (K == 0 ? B::kLead : 0);
      if constexpr (K == 0 && B::kLead) {
        ops.template at<U - 1, B::prev(0), B::kLast>();
        D[0] = mfma_bc<(U - 1) % 16>(ops.cur, X[B::lead()], D[0]);
      }
      const float xk = X[B::in(K)];
      static_for<0, kNC>([&](auto c) __attribute__((always_inline)) {
        constexpr int u = U + decltype(c)::value;
        ops.template at<u, decltype(c)::value == 0 && !(K == 0 && B::kLead) ? B::prev(K) : u - 1, B::kLast>();
        D[c] = mfma_bc<u % 16>(ops.cur, xk, D[c]);
      });
    }
  }
  __device__ __forceinline__ void store(float* X) {
    if constexpr (B::kCols > 0)
      static_for<0, B::kRows>([&](auto r) __attribute__((always_inline)) {
        X[B::out(decltype(r)::value)] = D[decltype(r)::value / 4][decltype(r)::value % 4];
      });
  }
};

__host__ __device__ constexpr int max_of(int a) { return a; }
template <class... T>
__host__ __device__ constexpr int max_of(int a, int b, T... r) {
  return max_of(a > b ? a : b, r...);
}

template <class... B>
__device__ __forceinline__ void blocks_mf(float* X, Ops& ops) {
  std::tuple<Acc<B>...> acc;
  std::apply(
      [&](auto&... b) __attribute__((always_inline)) {
        static_for<0, max_of(B::kCols...)>([&](auto k) __attribute__((always_inline)) {
          (b.template step<decltype(k)::value>(X, ops), ...);
        });
        (b.store(X), ...);
      },
      acc);
}

// sub-block B of step S of a J application at order P (lane_ops.h)
template <int P, int S, int B>
struct JSub {
  static constexpr int kD = lops::ju_degree(P, S, B);
  static constexpr int kCls = S & 1, kA = B & 1;
  static constexpr int kCols = lops::ju_cols(P, S, B), kRows = lops::ju_rows(P, S, B);
  static constexpr int kLead = lops::ju_lead(P, S, B);
  __host__ __device__ static constexpr int lead() { return kD * kD + lops::cls_member(kD, kCls, 0); }
  static constexpr int kLast = lops::ju(P, lops::ju_steps(P), 0, 0) - 1;
  __host__ __device__ static constexpr int u(int k) { return lops::ju(P, S, k, B); }
  __host__ __device__ static constexpr int prev(int k) { return u(k) - 1; }
  __host__ __device__ static constexpr int in(int k) {
    return kD * kD + lops::cls_member(kD, kCls, kA + lops::j_step(lops::cls_size(kD, kCls)) * k);
  }
  __host__ __device__ static constexpr int out(int r) {
    return kD * kD + lops::cls_member(kD, kCls, lops::j_first_row(kD, kCls, kA) +
                                                    lops::j_step(lops::cls_size(kD, kCls)) * r);
  }
};
// part T (cosine or sine) of block B of step M of the z translation
template <int P, int M, int B, int T>
struct ZBlk {
  static constexpr int kM = B == 0 ? M : P - M;
  static constexpr int kCols = kM >= T ? lops::zu_size(P, M, B) : 0;
  static constexpr int kRows = kCols, kLead = 0;
  __host__ __device__ static constexpr int lead() { return 0; }
  static constexpr int kLast = lops::zu(P, P / 2 + 1, 0, 0) - 1;
  __host__ __device__ static constexpr int u(int k) { return lops::zu(P, M, k, B); }
  // the instruction issued before column k: the sine parts skip the block of
  // order 0, beside which the one instruction of order P runs
  __host__ __device__ static constexpr int prev(int k) {
    if (T == 1 && M == 0) return -1;
    if (T == 1 && M == 1 && B == 0 && k == 0) return lops::zu(P, 0, 0, 1);
    return u(k) - 1;
  }
  __host__ __device__ static constexpr int in(int k) { return cidx(kM + k, kM, T); }
  __host__ __device__ static constexpr int out(int r) { return cidx(kM + r, kM, T); }
};

// X <- J X or J^T X on the matrix cores: per degree and parity class the two
// sub-blocks that hold the class block's nonzero entries times the lane's
// class members (lane_ops.h), degree n beside degree P - n, one class at a
// time.  The sub-blocks take 268 instructions per
// application at order 12, the whole class blocks 428 (half of their products
// with zeros).
template <int P>
__device__ __forceinline__ void japply_mf(float* X, Ops ops) {
  static_for<0, lops::ju_steps(P)>([&](auto sI) __attribute__((always_inline)) {
    constexpr int st = decltype(sI)::value;
    blocks_mf<JSub<P, st, 0>, JSub<P, st, 1>, JSub<P, st, 2>, JSub<P, st, 3>>(X, ops);
    // a few blocks at a time: bounded registers
    __builtin_amdgcn_sched_barrier(0);
  });
}

// (cos m g, sin m g), m = 1 .. P, of one lane's turn angle, from (c1, s1) =
// (cos g, sin g) by f_{m+1} = 2 cos g f_m - f_{m-1} in binary64, rounded to
// binary32 and kept in LDS for the turn back by the same angle: two orders to
// a 16-byte word, the words of a wave's lanes side by side.  (Held in
// registers they would spill; worked out again they are a tenth of the
// kernel's vector instructions.)
template <int P>
struct Turn {
  static constexpr int kWords = (P + 1) / 2;
  float c[P + 2], s[P + 2];
  __device__ __forceinline__ void make(double c1, double s1) {
    const double t = 2.0 * c1;
    double cp = 1.0, sp = 0.0, cc = c1, ss = s1;
#pragma unroll
    for (int m = 1; m <= P; ++m) {
      c[m] = (float)cc;
      s[m] = (float)ss;
      const double cn = t * cc - cp, sn = t * ss - sp;
      cp = cc;
      sp = ss;
      cc = cn;
      ss = sn;
    }
    c[P + 1] = s[P + 1] = 0.f;
  }
  __device__ __forceinline__ void put(float4* w) const {
#pragma unroll
    for (int i = 0; i < kWords; ++i) w[64 * i] = make_float4(c[2 * i + 1], s[2 * i + 1], c[2 * i + 2], s[2 * i + 2]);
  }
  __device__ __forceinline__ void get(const float4* w) {
    asm volatile("" ::: "memory");  // read from LDS, not from registers kept since put()
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
      const float4 v = w[64 * i];
      c[2 * i + 1] = v.x;
      s[2 * i + 1] = v.y;
      c[2 * i + 2] = v.z;
      s[2 * i + 2] = v.w;
    }
  }
};

// X <- Rz(-g) X in turns 1 and 2 of the translation, Rz(g) X in turns 3 and 4.
// The products to be rounded before the addition are named one by one (cosine
// terms fused on the way in, sine terms on the way back; at orders up to 4 the
// even orders m of turns 2 to 4 the other way round): left to the compiler, the
// choice changes with the code around it, and results in the eighth digit
// with it.
template <int P, int TURN>
__device__ __forceinline__ void rotz(float* X, const Turn<P>& g) {
  constexpr bool BACK = TURN > 2;
#pragma unroll
  for (int m = 1; m <= P; ++m) {
    const float c = g.c[m], s = g.s[m];
    const bool fuse_sin = BACK != (P <= 4 && TURN > 1 && m % 2 == 0);
#pragma unroll
    for (int n = m; n <= P; ++n) {
      const float a = X[cidx(n, m, 0)], b = X[cidx(n, m, 1)];
      const float u = BACK ? b : a, v = BACK ? a : b;  // the sum is c u + s v, the difference c v - s u
      const float sum = fuse_sin ? __builtin_fmaf(s, v, c * u) : __builtin_fmaf(c, u, s * v);
      const float dif = __builtin_fmaf(c, v, -(s * u));
      X[cidx(n, m, 0)] = BACK ? dif : sum;
      X[cidx(n, m, 1)] = BACK ? sum : dif;
    }
  }
}
// the turn by -g, whose cosines and sines go to w, and the turn back
template <int P, int TURN>
__device__ __forceinline__ void turn_in(float* X, double c1, double s1, float4* w) {
  Turn<P> g;
  g.make(c1, s1);
  g.put(w);
  rotz<P, TURN>(X, g);
}
template <int P, int TURN>
__device__ __forceinline__ void turn_back(float* X, const float4* w) {
  Turn<P> g;
  g.get(w);
  rotz<P, TURN>(X, g);
}

// the z-axis translation with the core products on the matrix cores: per
// order m the block A[m][d][n] (d, n = m .. P) times the lane's cosine and
// sine parts of order m (one operand table for both)
template <int P, class F>
__device__ __forceinline__ void ztrans_mf(float* X, const float* tab, int lane, const F& fac) {
  {
    const float in_base = fac.get(0);
    float w = in_base;
#pragma unroll
    for (int n = 1; n <= P; ++n) {
#pragma unroll
      for (int i = 0; i < 2 * n + 1; ++i) X[n * n + i] *= w;
      w *= in_base;
    }
  }
  // order m beside order P - m, the cosine parts, then the sine parts
  static_for<0, 2>([&](auto tI) __attribute__((always_inline)) {
    constexpr int T = decltype(tI)::value;
    Ops ops(tab, lane);
    static_for<0, P / 2 + 1>([&](auto mI) __attribute__((always_inline)) {
      constexpr int m = decltype(mI)::value;
      blocks_mf<ZBlk<P, m, 0, T>, ZBlk<P, m, 1, T>>(X, ops);
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  const float out_base = fac.get(1);
  float w = fac.get(2);
#pragma unroll
  for (int d = 0; d <= P; ++d) {
#pragma unroll
    for (int i = 0; i < 2 * d + 1; ++i) X[d * d + i] *= w;
    w *= out_base;
  }
}

// One halving exchange of the sum over the lanes, ND = ceil(NS / 2): dst[i]
// = src[i] of this lane and of its partner at lane distance D (lanes with
// bit D clear) or src[ND + i] of both (bit set); the upper half of an odd
// count is padded with zero.  Distances 32 and 16 are permlane swaps (the swap of (lower,
// upper) leaves each lane the two terms of its own sum), 8, 2 and 1 a DPP
// read of the partner, 4 two DPP shifts.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int NS, int D>
__device__ __forceinline__ void halve(const float* src, float* dst, int lane) {
  constexpr int ND = (NS + 1) / 2;
  const bool up = (lane & D) != 0;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const float lo = src[i];
    const float hi = ND + i < NS ? src[ND + i] : 0.f;
    if constexpr (D == 32 || D == 16) {
      const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false)
                             : __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
      dst[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else if constexpr (D == 4) {
      // row_shl:4 reads lane + 4, row_shr:4 lane - 4 (within rows of 16)
      const float t0 = lo + dpp<0x104>(lo), t1 = hi + dpp<0x114>(hi);
      dst[i] = up ? t1 : t0;
    } else {
      // the partner lane^D: row_ror:8, quad_perm [2,3,0,1], [1,0,3,2]
      constexpr int C = D == 8 ? 0x128 : D == 2 ? 0x4E : 0xB1;
      const float send = up ? lo : hi, keep = up ? hi : lo;
      dst[i] = keep + dpp<C>(send);
    }
    if ((i & 7) == 7) __builtin_amdgcn_sched_barrier(0);  // a few in flight: bounded registers
  }
}

__device__ __forceinline__ int level_of3(const LevelView& lv, int64_t gid) {
  int l = 0;
  while (l < lv.L && gid >= lv.gofs[l + 1]) ++l;
  return l;
}

// Waves per SIMD, as the registers allow (two at 12 with a few values parked
// in LDS; at 13 172 would spill: 75.2 ms against 47.9 with one wave on the
// cloud below).
// What bounds the kernel: instruction issue, matrix and vector instructions
// never running together.  Measured on 2^22 Plummer points (5 levels, theta
// 0.6, 194 million pairs), M2L in ms: order 4 4.2, 6 7.5, 8 11.7, 10 18.1, 11
// 22.0, 12 27.5 (103 TFLOP/s by the dense count of 14,638 flops a
// pair), 13 46.2, 14 54.6; with whole class blocks for J and the turns' angles
// worked out twice 4.6, 8.7, 14.7, 23.5, 29.2, 37.8, 58.2 and 69.3.
template <int P>
struct LaneCfg {
  static constexpr int kWaves = P <= 6 ? 4 : P <= 8 ? 3 : P <= 12 ? 2 : 1;
  // at order 12 15 values would spill without (28.4 ms instead of 27.5 on the
  // cloud above); elsewhere the LDS traffic only costs (1 to 5 %)
  static constexpr bool kPark = P == 12;
};

// SHARE, RUNS: how the targets are dealt out (m2l_queue.h); template arguments,
// as a scalar more in the loop's registers spills at the highest orders
template <int P, bool SHARE, bool RUNS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LaneCfg<P>::kWaves, LaneCfg<P>::kWaves))) void
k_m2l_lane(LevelView lv, const float* __restrict__ ltab, const int* __restrict__ pos, const float* __restrict__ Mf,
           double* __restrict__ Lx, int64_t ntarget, const int32_t* __restrict__ order, int* __restrict__ queue) {
  constexpr int NT = (P + 1) * (P + 1);
  constexpr int S = tl::stride(P);
  constexpr int SD = lops::dense_stride(P);
  constexpr int NF = lvl(NT, 6);  // values a lane holds after the exchanges
  constexpr int GJ = 64 * lops::groups(lops::n_j(P));  // table: J, J^T, z core
  __shared__ float tabs[lops::table_floats(P)];
  // the turn angles' cosines and sines: two angles per lane (12 KB per wave at
  // order 12; with the tables and the parked values 80 KB per block, so that two
  // blocks just fit on a CU)
  constexpr int TW = 64 * Turn<P>::kWords;
  __shared__ float4 turns[P > 0 ? 4 * 2 * TW : 1];
  // values that a lane parks while the translation runs, where they would
  // spill: the sums over the batches and the polar angle; the distance factors
  constexpr bool PK = LaneCfg<P>::kPark;
  __shared__ double parkd[PK ? (NF + 2) * 256 : SHARE ? NF * 256 : 1];
  __shared__ float parkf[PK ? 3 * 256 : 1];
  for (int i = threadIdx.x; i < lops::table_floats(P); i += blockDim.x) tabs[i] = ltab[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  float4* wb = turns + (threadIdx.x >> 6) * 2 * TW + (P > 0 ? lane : 0);  // beta, then alpha
  float4* wa = wb + TW;
  m2lq::Cursor<RUNS> cur;
  const int wave = SHARE ? m2lq::uniform((int)(threadIdx.x >> 6)) : 0;
  for (;;) {
    const int64_t kq = SHARE ? (int64_t)blockIdx.x : cur.next(queue, ntarget, lane);
    if (kq >= ntarget) break;
    // the target's data are the same in all lanes: kept in scalar registers
    const int64_t gid = lv.gofs[1] + m2lq::uniform(order[kq]);
    const int l = level_of3(lv, gid);
    const int64_t bi = gid - lv.gofs[l];
    const double* geo = lv.geom[l];
    const double cix = m2lq::uniform(geo[bi * 10 + 6]), ciy = m2lq::uniform(geo[bi * 10 + 7]);
    const double ciz = m2lq::uniform(geo[bi * 10 + 8]), rt_ = m2lq::uniform(geo[bi * 10 + 9]);
    const double rt = rt_ > 0.0 ? rt_ : 1.0;
    const int32_t* wrow = lv.w_idx[l] + m2lq::uniform(lv.w_off[l][bi]);
    const int ne = (int)m2lq::uniform(lv.w_off[l][bi + 1] - lv.w_off[l][bi]);
    const float* Mlev = Mf + (size_t)lv.gofs[l] * SD;
    m2lq::Kept<double, NF + 2, PK> acc(parkd + threadIdx.x, 256);  // the sums, ca, sa
    m2lq::Kept<float, 3, PK> fac(parkf + threadIdx.x, 256);        // in_base, out_base, out_mult
#pragma unroll
    for (int i = 0; i < NF; ++i) acc.put(i, 0.0);

    // the next batch's source indexes are loaded while this batch runs
    const int b0 = 64 * wave, bs = 64 * (SHARE ? 4 : 1);
    int32_t jn = ne > 0 ? wrow[b0 + lane < ne ? b0 + lane : 0] : 0;
    for (int eb = b0; eb < ne; eb += bs) {
      const int e = eb + lane;
      const bool valid = e < ne;
      const int64_t j = jn;
      jn = wrow[e + bs < ne ? e + bs : 0];
      const double dx = geo[j * 10 + 6] - cix, dy = geo[j * 10 + 7] - ciy, dz = geo[j * 10 + 8] - ciz;
      const double rs = geo[j * 10 + 9] > 0.0 ? geo[j * 10 + 9] : 1.0;
      const double rxy2 = dx * dx + dy * dy;
      const double irho = m2lq::rsqrt0(rxy2 + dz * dz), irxy = m2lq::rsqrt0(rxy2);
      const double ca = dz * irho, sa = rxy2 * irxy * irho;
      const double cb = rxy2 > 0.0 ? dx * irxy : 1.0, sb = dy * irxy;
      // a lane past the end of the list translates the first source with zero factors
      fac.put(0, valid ? (float)(rs * irho) : 0.f);
      fac.put(1, valid ? (float)(rt * irho) : 0.f);
      fac.put(2, valid ? (float)irho : 0.f);
      acc.put(NF, ca);
      acc.put(NF + 1, sa);

      float X[NT];
      const float4* src = (const float4*)(Mlev + (size_t)j * SD);
#pragma unroll
      for (int q = 0; q < SD / 4; ++q) {
        const float4 v = src[q];
        if (4 * q + 0 < NT) X[4 * q + 0] = v.x;
        if (4 * q + 1 < NT) X[4 * q + 1] = v.y;
        if (4 * q + 2 < NT) X[4 * q + 2] = v.z;
        if (4 * q + 3 < NT) X[4 * q + 3] = v.w;
      }

      // the steps are kept apart in the schedule (interleaving them only
      // raises the number of live values)
#define FMM_STEP(x)                      \
  x;                                     \
  __builtin_amdgcn_sched_barrier(0)
      // the first operands of a quarter turn are loaded before the z-turn
      // ahead of it
      const float *tJ = tabs, *tJT = tabs + GJ;
      FMM_STEP(Ops o1(tJT, lane));
      FMM_STEP((turn_in<P, 1>(X, cb, sb, wb)));
      FMM_STEP(japply_mf<P>(X, o1));
      FMM_STEP(Ops o2(tJ, lane));
      FMM_STEP((turn_in<P, 2>(X, acc.get(NF), acc.get(NF + 1), wa)));
      FMM_STEP(japply_mf<P>(X, o2));
      FMM_STEP(ztrans_mf<P>(X, tabs + 2 * GJ, lane, fac));
      FMM_STEP(japply_mf<P>(X, Ops(tJT, lane)));
      FMM_STEP(Ops o4(tJ, lane));
      FMM_STEP((turn_back<P, 3>(X, wa)));
      FMM_STEP(japply_mf<P>(X, o4));
      FMM_STEP((turn_back<P, 4>(X, wb)));
#undef FMM_STEP

      // sum over the 64 lanes: six halving exchanges; at the exchange with
      // lane distance d the lanes with bit d clear keep the lower half
      float h1[lvl(NT, 1)], h2[lvl(NT, 2)], h3[lvl(NT, 3)], h4[lvl(NT, 4)], h5[lvl(NT, 5)], h6[lvl(NT, 6)];
      halve<NT, 32>(X, h1, lane);
      halve<lvl(NT, 1), 16>(h1, h2, lane);
      halve<lvl(NT, 2), 8>(h2, h3, lane);
      halve<lvl(NT, 3), 4>(h3, h4, lane);
      halve<lvl(NT, 4), 2>(h4, h5, lane);
      halve<lvl(NT, 5), 1>(h5, h6, lane);
#pragma unroll
      for (int i = 0; i < NF; ++i) acc.put(i, acc.get(i) + (double)h6[i]);
    }
    if constexpr (SHARE) {  // the waves' sums, in wave order
      if constexpr (!PK)
#pragma unroll
        for (int i = 0; i < NF; ++i) parkd[i * 256 + threadIdx.x] = acc.get(i);
      __syncthreads();
      if (threadIdx.x >= 64) return;
      for (int w = 64; w < 256; w += 64)
#pragma unroll
        for (int i = 0; i < NF; ++i) acc.put(i, acc.get(i) + parkd[i * 256 + w + lane]);
    }
    // lane's values: standard index base + i, where each exchange added the
    // kept half's offset; entries past a half's end are padding
    int base = 0, len = NT;
#pragma unroll
    for (int sidx = 1; sidx <= 6; ++sidx) {
      const int half = lvl(NT, sidx);
      const int dist = 64 >> sidx;
      if (lane & dist) {
        base += half;
        len = len - half > 0 ? len - half : 0;
      } else {
        len = len < half ? len : half;
      }
    }
    double* dst = Lx + (size_t)gid * S;
    const double irt = 1.0 / rt;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      if (i >= len) continue;
      const int k = base + i;
      const int n = deg_of(k);
      double v = acc.get(i);
      for (int q = 0; q < n; ++q) v *= irt;
      dst[pos[k]] = v;
    }
    if constexpr (SHARE) return;
  }
}

// The binary32 multipoles of levels 1..L for this kernel, from the binary64
// ones (tile layout, S per box): standard order, scaled by r^-n (r the box
// radius, 1 for a box of zero extent; the same products as for the tile
// kernel's copy), lops::dense_stride(P) floats per box with a zero tail.
template <int P>
__global__ void k_scale_lane(LevelView lv, int S, const int* __restrict__ pos, const double* __restrict__ Mx,
                             float* __restrict__ Mf, int64_t nbox_total) {
  constexpr int NT = (P + 1) * (P + 1), SD = lops::dense_stride(P);
  const int64_t gid = 1 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (gid >= nbox_total) return;
  int l = 1;
  while (l < lv.L && gid >= lv.gofs[l + 1]) ++l;
  const double r = lv.geom[l][(gid - lv.gofs[l]) * 10 + 9];
  const double is = r > 0.0 ? 1.0 / r : 1.0;
  for (int k = threadIdx.x & 63; k < SD; k += 64) {
    float v = 0.f;
    if (k < NT) {
      const int n = deg_of(k);
      double d = Mx[(size_t)gid * S + pos[k]];
      for (int q = 0; q < n; ++q) d *= is;
      v = (float)d;
    }
    Mf[(size_t)gid * SD + k] = v;
  }
}

__global__ void k_start_queue_l(int* queue) {
  if (threadIdx.x < m2lq::kXcds) queue[threadIdx.x] = 0;
}

template <int P>
void launch_one_lane(const Tree& t, const Tables& tb, const double* Mx, double* Lx, hipStream_t s) {
  const int64_t ntarget = t.nbox_total - 1;
  if (ntarget <= 0) return;
  float* Mf = (float*)dalloc((size_t)t.nbox_total * lops::dense_stride(P) * sizeof(float), s);
  k_scale_lane<P><<<(unsigned)((ntarget + 3) / 4), 256, 0, s>>>(t.view(), tb.stride, tb.pos, Mx, Mf, t.nbox_total);
  HIPCHECK(hipGetLastError());
  if (ntarget <= m2lq::kShareLane) {
    k_m2l_lane<P, true, false><<<(unsigned)ntarget, 256, 0, s>>>(t.view(), tb.lane, tb.pos, Mf, Lx, ntarget,
                                                                  t.m2l_order, nullptr);
    HIPCHECK(hipGetLastError());
    dfree(Mf, s);
    return;
  }
  static const int grid_max = [] {
    int dev = 0, ncu = 0, per = 0;
    HIPCHECK(hipGetDevice(&dev));
    HIPCHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    HIPCHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_m2l_lane<P, false, false>, 256, 0));
    return ncu * (per > 0 ? per : 1);
  }();
  const int64_t need = (ntarget + 3) / 4;
  const unsigned grid = (unsigned)(need < grid_max ? need : grid_max);
  int* queue = (int*)dalloc(m2lq::kXcds * sizeof(int), s);
  k_start_queue_l<<<1, 64, 0, s>>>(queue);
  HIPCHECK(hipGetLastError());
  if (ntarget >= kM2LSiblingsMin)
    k_m2l_lane<P, false, true><<<grid, 256, 0, s>>>(t.view(), tb.lane, tb.pos, Mf, Lx, ntarget, t.m2l_order, queue);
  else
    k_m2l_lane<P, false, false><<<grid, 256, 0, s>>>(t.view(), tb.lane, tb.pos, Mf, Lx, ntarget, t.m2l_order, queue);
  HIPCHECK(hipGetLastError());
  dfree(queue, s);
  dfree(Mf, s);
}

}  // namespace

// mixed-precision M2L with this kernel from the binary64 multipoles Mx (tile
// layout); false above order 14, where the 16x16 tile kernel is as fast
bool launch_m2l_lane32(const Tree& t, const Tables& tb, const double* Mx, double* Lx, hipStream_t s) {
  switch (tb.p) {
    case 0: launch_one_lane<0>(t, tb, Mx, Lx, s); break;
    case 1: launch_one_lane<1>(t, tb, Mx, Lx, s); break;
    case 2: launch_one_lane<2>(t, tb, Mx, Lx, s); break;
    case 3: launch_one_lane<3>(t, tb, Mx, Lx, s); break;
    case 4: launch_one_lane<4>(t, tb, Mx, Lx, s); break;
    case 5: launch_one_lane<5>(t, tb, Mx, Lx, s); break;
    case 6: launch_one_lane<6>(t, tb, Mx, Lx, s); break;
    case 7: launch_one_lane<7>(t, tb, Mx, Lx, s); break;
    case 8: launch_one_lane<8>(t, tb, Mx, Lx, s); break;
    case 9: launch_one_lane<9>(t, tb, Mx, Lx, s); break;
    case 10: launch_one_lane<10>(t, tb, Mx, Lx, s); break;
    case 11: launch_one_lane<11>(t, tb, Mx, Lx, s); break;
    case 12: launch_one_lane<12>(t, tb, Mx, Lx, s); break;
    case 13: launch_one_lane<13>(t, tb, Mx, Lx, s); break;
    case 14: launch_one_lane<14>(t, tb, Mx, Lx, s); break;
    default: return false;
  }
  return true;
}

}  // namespace fmm
