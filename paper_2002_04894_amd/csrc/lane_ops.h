// Operand order of the per-lane M2L kernel (m2l_lane.hip) on the 16-block
// 4x4x1 matrix instruction, shared by the kernel and by the host code that
// packs its operator tables.
//
// Each lane holds one pair's expansion; a fixed operator block B (s x s) acts
// on s of the lane's coefficients as a sequence of instructions, one per
// (input column k, output chunk c of 4 rows): D_c += B[4c .. 4c+3][k] * x_k.
// The 4 operator values of an instruction are the A operand of one block,
// broadcast to all 16 blocks, so 16 consecutive instructions take theirs from
// one register: the table holds, per group of 16 instructions, 64 values,
// value 4 * (u mod 16) + i = row i of instruction u (zero past the block).
// The instructions are numbered in the order in which the kernel issues them
// (ju, zu below), so that one register holds the operands of all blocks in
// flight.
//
// Blocks, in order:
//   J or J^T: per degree n, per parity class cls (0: n+1 members, 1: n), the
//             class members in standard order (the quarter turn about x
//             keeps the classes apart).  The turn also carries reflections in
//             y into reflections in z, so half the entries of a class block
//             vanish: a class of more than four members runs as two
//             sub-blocks (j_rows below);
//   z core:   per order m, rows d and columns n = m .. P (one table for the
//             cosine and the sine parts, which share it).  Orders m and p - m
//             run in lock-step.
#pragma once

namespace fmm {
namespace lops {

// 0 / 1: the two classes of the standard index i within a degree (c_m at
// i = 2m-1, s_m at i = 2m) that the quarter turn about x keeps apart
__host__ __device__ constexpr int parity_cls(int i) {
  return i == 0 ? 0 : ((((i + 1) >> 1) + ((i & 1) ? 0 : 1)) & 1);
}
__host__ __device__ constexpr int cls_size(int n, int cls) { return cls == 0 ? n + 1 : n; }
// r-th member (standard index within degree n) of class cls
__host__ __device__ constexpr int cls_member(int n, int cls, int r) {
  for (int i = 0; i < 2 * n + 1; ++i)
    if (parity_cls(i) == cls && r-- == 0) return i;
  return -1;
}
__host__ __device__ constexpr int chunks(int s) { return (s + 3) / 4; }
// first instruction of block (n, cls) of a J application, and of order m of
// the z translation at expansion order p (its blocks have p + 1 - m rows)
__host__ __device__ constexpr int j_offset(int n, int cls) {
  int u = 0;
  for (int a = 0; a < n; ++a)
    for (int c = 0; c < 2; ++c) u += cls_size(a, c) * chunks(cls_size(a, c));
  return cls == 0 ? u : u + cls_size(n, 0) * chunks(cls_size(n, 0));
}
__host__ __device__ constexpr int z_offset(int p, int m) {
  int u = 0;
  for (int a = 0; a < m; ++a) u += (p + 1 - a) * chunks(p + 1 - a);
  return u;
}
// Entry (r, k) of the class block (n, cls) of J or J^T is zero unless
// r + k + n + cls is even: member r is even under y -> -y iff r is even, and
// under z -> -z iff r + n + cls is, and the quarter turn exchanges the two.  A
// class of more than four members is split by the parity a of its columns:
// sub-block a takes the columns a, a + 2, ... and gives the rows first_row,
// first_row + 2, ...; up to four members share one chunk of rows, where a
// split saves nothing.
__host__ __device__ constexpr bool j_split(int s) { return s > 4; }
__host__ __device__ constexpr int j_step(int s) { return j_split(s) ? 2 : 1; }
__host__ __device__ constexpr int j_cols(int s, int a) { return j_split(s) ? (s + 1 - a) / 2 : (a == 0 ? s : 0); }
__host__ __device__ constexpr int j_first_row(int n, int cls, int a) {
  return j_split(cls_size(n, cls)) ? (a + n + cls) & 1 : 0;
}
__host__ __device__ constexpr int j_rows(int n, int cls, int a) {
  return j_split(cls_size(n, cls)) ? (cls_size(n, cls) + 1 - j_first_row(n, cls, a)) / 2
                                   : j_cols(cls_size(n, cls), a);
}
// The rows of sub-block 1 begin behind a column that vanishes.  Where the first
// entry of a row is a short binary fraction (in the first chunk of rows, at
// these classes: 3/4, 1/2, -5/8, 9/16, ...), its product often lies halfway
// between two binary32 values, and the vanishing entry before it, about 1e-21
// as tabulated, decides the rounding.  That one instruction is kept, so that
// every rounding is that of the whole block: 40 of 1,500 instructions per batch at
// order 12, for results that differ in the tenth digit without.  Which classes
// have such entries was read off the tables of orders up to 14.
__host__ __device__ constexpr bool j_lead(int n, int cls) { return ((n + cls) & 1) == 0 || n == 6; }
// instructions of one J application and of the z translation (per part)
__host__ __device__ constexpr int n_j(int p) { return j_offset(p + 1, 0); }
__host__ __device__ constexpr int n_z(int p) { return z_offset(p, p + 1); }
__host__ __device__ constexpr int groups(int u) { return (u + 15) / 16; }
// The table reserves n_j instructions for a J application, one per (column,
// output chunk) of whole class blocks; its sub-blocks need about half of them.
//
// Step t of a J application at order p (t = 0 .. 2 (p / 2) + 1) runs class t & 1
// of degrees t / 2 (sub-blocks b = 0, 1 for column parity b) and p - t / 2
// (b = 2, 3 for column parity b - 2, absent unless p - t / 2 > t / 2), column
// by column: four or five accumulator chains in flight in most steps, which
// covers the latency of the instruction and leaves registers for the
// expansion.
__host__ __device__ constexpr int ju_steps(int p) { return 2 * (p / 2 + 1); }
__host__ __device__ constexpr int ju_degree(int p, int t, int b) {
  return b < 2 ? t / 2 : (p - t / 2 > t / 2 ? p - t / 2 : -1);
}
__host__ __device__ constexpr int ju_cols(int p, int t, int b) {
  const int d = ju_degree(p, t, b);
  return d < 0 ? 0 : j_cols(cls_size(d, t & 1), b & 1);
}
__host__ __device__ constexpr int ju_rows(int p, int t, int b) {
  return ju_cols(p, t, b) == 0 ? 0 : j_rows(ju_degree(p, t, b), t & 1, b & 1);
}
// 1 if sub-block b of step t begins with the instruction of the class's column
// 0 on its first chunk of rows (j_lead)
__host__ __device__ constexpr int ju_lead(int p, int t, int b) {
  const int d = ju_degree(p, t, b);
  return d >= 0 && (b & 1) && ju_cols(p, t, b) > 0 && j_lead(d, t & 1) ? 1 : 0;
}
// number of the first instruction of column k of sub-block b in step t
__host__ __device__ constexpr int ju(int p, int t, int k, int b) {
  int u = 0;
  for (int s = 0; s < t; ++s)
    for (int c = 0; c < 4; ++c) u += ju_lead(p, s, c) + ju_cols(p, s, c) * chunks(ju_rows(p, s, c));
  for (int c = 0; c < 4; ++c) {
    const int cols = ju_cols(p, t, c), done = c < b ? k + 1 : k;
    u += (done > 0 ? ju_lead(p, t, c) : 0) + (cols < done ? cols : done) * chunks(ju_rows(p, t, c));
  }
  return u;
}
// Step m of the z translation runs the blocks of orders m (b = 0) and p - m
// (b = 1, absent unless p - m > m), p + 1 - order rows each, once for the
// cosine and once for the sine parts.
__host__ __device__ constexpr int zu_size(int p, int m, int b) {
  return b == 0 ? p + 1 - m : (p - m > m ? m + 1 : 0);
}
__host__ __device__ constexpr int zu(int p, int m, int k, int b) {
  int u = 0;
  for (int s = 0; s < m; ++s)
    for (int c = 0; c < 2; ++c) u += zu_size(p, s, c) * chunks(zu_size(p, s, c));
  for (int c = 0; c < 2; ++c) {
    const int cols = zu_size(p, m, c), done = c < b ? k + 1 : k;
    u += (cols < done ? cols : done) * chunks(cols);
  }
  return u;
}
// floats per box of the binary32 multipoles the per-lane kernel reads: the
// (p+1)^2 coefficients in the standard order, padded to whole 16-byte loads
__host__ __device__ constexpr int dense_stride(int p) { return ((p + 1) * (p + 1) + 3) & ~3; }
// table floats: J, J^T, z core, each padded to whole groups
__host__ __device__ constexpr int table_floats(int p) { return 64 * (2 * groups(n_j(p)) + groups(n_z(p))); }

// ---- the binary64 per-quad M2L kernel (m2l_quad.hip) on v_mfma_f64_4x4x4f64 ----
//
// A wave takes 16 pairs; lane 16 k + q holds phase k (0..3) of pair q.  Per
// degree d the coefficients form two blocks indexed by the order m = 0..d:
// block 0 holds c_m for even m and s_m for odd m, block 1 the others (its
// member 0, s_0, is a zero slot) -- the two classes that the quarter turn
// about x keeps apart, ordered by m.  Entry (m', m) of a block is zero unless
// m' + m + d + x is even (the reflections in y and z, as above), so the
// members are dealt to the registers by parity (qorder): of each eight orders
// the even ones fill one register and the odd ones the next, or, where at most
// four of the eight exist, all share one.  A part (output register c, input
// register g) whose entries all vanish is left out.  The cosine and sine parts
// of (d, m) share a lane and register index.  An exchange of the two halves of
// the wave between an even and an odd register sorts them by order again: the
// lower four orders of the eight in the first, as in a shared register, the
// upper four in the second, so that all degrees of an order share a lane.  The
// operand of instruction u is 16 values, row i and column k of its 4x4 part at
// 16 u + 4 k + i (the lane layout of the instruction: lane 16 k + 4 b + i holds
// A[i][k] of block b, for every b).
__host__ __device__ constexpr int qreg(int d) { return d / 4 + 1; }
// first register of block (d, x)
__host__ __device__ constexpr int qbase(int d, int x) {
  int r = 0;
  for (int a = 0; a < d; ++a) r += 2 * qreg(a);
  return r + x * qreg(d);
}
__host__ __device__ constexpr int nq(int p) { return qbase(p + 1, 0); }
// standard index within degree d of member m of block x, or -1 for a zero slot
__host__ __device__ constexpr int qmember(int d, int x, int m) {
  if (m > d) return -1;
  if ((m & 1) == x) return m == 0 ? 0 : 2 * m - 1;  // c_m
  return m == 0 ? -1 : 2 * m;                       // s_m
}
// order of the member in phase k of register g of a block of degree d (none
// if above d), and the position of order e = 0..3 of a shared register
__host__ __device__ constexpr int qshared(int k) { return 2 * (k & 1) + (k >> 1); }
__host__ __device__ constexpr bool qpaired(int d, int g) { return d + 1 - 8 * (g / 2) > 4; }
__host__ __device__ constexpr int qorder(int d, int g, int k) {
  return 8 * (g / 2) + (qpaired(d, g) ? 2 * k + (g & 1) : qshared(k));
}
// whether part (input register g, output register c) of block (d, x) holds
// nonzero entries, and its rank among those that do
__host__ __device__ constexpr bool qpart(int d, int x, int g, int c) {
  for (int k = 0; k < 4; ++k)
    for (int i = 0; i < 4; ++i) {
      const int m = qorder(d, g, k), r = qorder(d, c, i);
      if (m >= x && r >= x && m <= d && r <= d && ((m + r + d + x) & 1) == 0) return true;
    }
  return false;
}
__host__ __device__ constexpr int qpart_rank(int d, int x, int g, int c) {
  int n = 0;
  for (int a = 0; a < g; ++a)
    for (int b = 0; b < qreg(d); ++b) n += qpart(d, x, a, b) ? 1 : 0;
  for (int b = 0; b < c; ++b) n += qpart(d, x, g, b) ? 1 : 0;
  return n;
}
// first instruction of block (d, x) in one J application, were all parts of
// whole blocks kept
__host__ __device__ constexpr int qj_offset(int d, int x) {
  int u = 0;
  for (int a = 0; a < d; ++a) u += 2 * qreg(a) * qreg(a);
  return u + x * qreg(d) * qreg(d);
}
__host__ __device__ constexpr int qj_count(int p) { return qj_offset(p + 1, 0); }
// z-translation core A[m][d][n] for m = 0 .. p + 1 (order p + 1 all zero: the
// slot of the lanes whose order exceeds p)
__host__ __device__ constexpr int qcore_doubles(int p) { return (p + 2) * (p + 1) * (p + 1); }
// whether the table holds J^T beside J: where both fit in 160 KB of LDS with
// the core (orders up to 18); above, the kernel reads J^T from J transposed
__host__ __device__ constexpr bool qtable_has_jt(int p) {
  return (2 * 16 * qj_count(p) + qcore_doubles(p)) * 8 <= 160 * 1024;
}
// table: J (16 values per instruction), J^T in the same form if it fits, then
// the z-translation core
__host__ __device__ constexpr int qtable_doubles(int p) {
  return (qtable_has_jt(p) ? 2 : 1) * 16 * qj_count(p) + qcore_doubles(p);
}

// The parts that are kept: first instruction of block (d, x), their number
__host__ __device__ constexpr int qp_offset(int d, int x) {
  int u = 0;
  for (int a = 0; a <= d; ++a)
    for (int b = 0; b < (a < d ? 2 : x); ++b) u += qpart_rank(a, b, qreg(a), 0);
  return u;
}
__host__ __device__ constexpr int qp_count(int p) { return qp_offset(p + 1, 0); }
// Threads of a block (one block per CU): two waves per SIMD up to order 15,
// where the registers allow it, one above.
__host__ __device__ constexpr int qthreads(int p) { return p <= 15 ? 512 : 256; }
// values a lane holds of the sum over a batch's 16 pairs
__host__ __device__ constexpr int qsums(int p) { return (nq(p) + 15) / 16; }
// bytes of LDS beside the tables: six values and the sums parked by each
// lane, a word for each (register, phase)
__host__ __device__ constexpr int qpark_bytes(int p) { return (6 + qsums(p)) * qthreads(p) * 8 + nq(p) * 16; }
// the tables: J (16 values per instruction), J^T in the same form where it
// fits beside the rest (orders up to 18; above, J^T is read from J
// transposed), the z-translation core
__host__ __device__ constexpr bool qp_has_jt(int p) {
  return (2 * 16 * qp_count(p) + qcore_doubles(p)) * 8 + qpark_bytes(p) <= 160 * 1024;
}
__host__ __device__ constexpr int qp_doubles(int p) {
  return (qp_has_jt(p) ? 2 : 1) * 16 * qp_count(p) + qcore_doubles(p);
}

}  // namespace lops
}  // namespace fmm
