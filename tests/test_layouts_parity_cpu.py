"""The parity split of the quarter turn in the operand layouts of the M2L
kernels (paper_2002_04894_amd/csrc/lane_ops.h), compiled for the host with
g++: every entry of a class block that the split calls nonzero is taken by
exactly one instruction row, the instruction numbers of a kernel's steps are
consecutive in the order of issue and stay inside the reserved table, and the
entries called zero are zero in the quarter turn itself (worked out here from
the rotated harmonics, in NumPy).
"""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INC = os.path.join(ROOT, "paper_2002_04894_amd", "csrc")

LANE = r"""
#define __host__
#define __device__
#include <cstdio>
#include <map>
#include <tuple>
#include "lane_ops.h"
using namespace fmm::lops;
int main() {
  int fails = 0;
  for (int p = 0; p <= 20; ++p) {
    std::map<std::tuple<int, int, int, int>, int> seen;
    int u = 0;
    for (int t = 0; t < ju_steps(p); ++t)
      for (int k = 0; k <= p; ++k)
        for (int b = 0; b < 4; ++b) {
          if (k >= ju_cols(p, t, b)) continue;
          const int n = ju_degree(p, t, b), cls = t & 1, rows = ju_rows(p, t, b), st = j_step(cls_size(n, cls));
          fails += ju(p, t, k, b) != u;
          u += chunks(rows) + (k == 0 ? ju_lead(p, t, b) : 0);
          for (int r = 0; r < rows; ++r)
            ++seen[{n, cls, j_first_row(n, cls, b & 1) + st * r, (b & 1) + st * k}];
        }
    fails += u != ju(p, ju_steps(p), 0, 0) || u > n_j(p);
    for (int n = 0; n <= p; ++n)
      for (int cls = 0; cls < 2; ++cls)
        for (int r = 0; r < cls_size(n, cls); ++r)
          for (int k = 0; k < cls_size(n, cls); ++k) {
            const int want = ((r + k + n + cls) & 1) == 0, got = seen.count({n, cls, r, k}) ? seen[{n, cls, r, k}] : 0;
            fails += got > 1 || (want && got != 1);
          }
    for (auto& e : seen) fails += std::get<2>(e.first) >= cls_size(std::get<0>(e.first), std::get<1>(e.first));
    u = 0;
    for (int m = 0; m <= p / 2; ++m)
      for (int k = 0; k <= p; ++k)
        for (int b = 0; b < 2; ++b) {
          if (k >= zu_size(p, m, b)) continue;
          fails += zu(p, m, k, b) != u;
          u += chunks(zu_size(p, m, b));
        }
    fails += u != n_z(p) || u != zu(p, p / 2 + 1, 0, 0);
  }
  std::printf("%d failures\n", fails);
  return fails != 0;
}
"""


QUAD = r"""
#define __host__
#define __device__
#include <cstdio>
#include <set>
#include <utility>
#include "lane_ops.h"
using namespace fmm::lops;
int main() {
  int fails = 0;
  for (int p = 0; p <= 20; ++p) {
    int u = 0;
    for (int d = 0; d <= p; ++d)
      for (int x = 0; x < 2; ++x) {
        // every order 0..d in exactly one (register, phase)
        std::set<int> orders;
        for (int g = 0; g < qreg(d); ++g)
          for (int k = 0; k < 4; ++k) {
            const int m = qorder(d, g, k);
            if (m <= d) fails += !orders.insert(m).second;
            // the exchange of wave halves sorts a pair of registers by order
            const int e = 4 * g + qshared(k);
            if (qpaired(d, g)) {
              const int src = (g & ~1) + (k >> 1), ph = 2 * (g & 1) + (k & 1);
              fails += qorder(d, src, ph) != e;
            } else {
              fails += m != e;
            }
          }
        fails += (int)orders.size() != d + 1;
        // kept parts: numbered without gaps, in order; the others hold no nonzero entry
        fails += qp_offset(d, x) != u;
        for (int g = 0; g < qreg(d); ++g)
          for (int c = 0; c < qreg(d); ++c) {
            bool any = false;
            for (int k = 0; k < 4; ++k)
              for (int i = 0; i < 4; ++i) {
                const int m = qorder(d, g, k), r = qorder(d, c, i);
                any = any || (qmember(d, x, m) >= 0 && qmember(d, x, r) >= 0 && (m + r + d + x) % 2 == 0);
              }
            fails += any != qpart(d, x, g, c);
            fails += qpart(d, x, g, c) != qpart(d, x, c, g);
            if (any) fails += qp_offset(d, x) + qpart_rank(d, x, g, c) != u++;
          }
      }
    fails += qp_count(p) != u;
    fails += qp_has_jt(p) != (p <= 18) || qp_doubles(p) * 8 + qpark_bytes(p) > 160 * 1024;
  }
  std::printf("%d failures\n", fails);
  return fails != 0;
}
"""


def run_host(tmp_path, program):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(program)
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", INC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout[-2000:]


@pytest.mark.parametrize("program", [LANE, QUAD], ids=["lane", "quad"])
def test_split_layouts(tmp_path, program):
    run_host(tmp_path, program)


def harmonics(p, v):
    """Schmidt semi-normalised real solid harmonics of degrees 0..p at the
    points v, per degree in the order c_0, c_1, s_1, ..."""
    x, y, z = v.T
    r2 = x * x + y * y + z * z
    g = {(0, 0): np.ones_like(x) + 0j}
    for m in range(p + 1):
        if m > 0:
            g[m, m] = math.sqrt((2 * m - 1) / (2 * m)) * (x + 1j * y) * g[m - 1, m - 1]
        if m < p:
            g[m + 1, m] = math.sqrt(2 * m + 1) * z * g[m, m]
        for n in range(m + 2, p + 1):
            g[n, m] = ((2 * n - 1) * z * g[n - 1, m] - math.sqrt((n + m - 1) * (n - m - 1)) * r2 * g[n - 2, m]) / \
                math.sqrt((n + m) * (n - m))
    return [np.stack([g[n, 0].real] + [f for m in range(1, n + 1)
                                       for f in (math.sqrt(2) * g[n, m].real, math.sqrt(2) * g[n, m].imag)], axis=1)
            for n in range(p + 1)]


def test_quarter_turn_zeros():
    """J of degree n by least squares over random directions (K: (x, y, z) ->
    (x, z, -y)); the entries that the layouts drop vanish to the solver's
    rounding: 1e-9 stands between it (about 1e-12) and the smallest kept
    entries that matter."""
    p = 10
    v = np.random.default_rng(0).standard_normal((400, 3))
    v /= np.linalg.norm(v, axis=1)[:, None]
    rotated = harmonics(p, np.stack([v[:, 0], v[:, 2], -v[:, 1]], axis=1))
    for n, (a, b) in enumerate(zip(harmonics(p, v), rotated)):
        J = np.linalg.lstsq(a, b, rcond=None)[0].T
        order = [(i + 1) // 2 for i in range(2 * n + 1)]
        sine = [i > 0 and i % 2 == 0 for i in range(2 * n + 1)]
        for i in range(2 * n + 1):
            for j in range(2 * n + 1):
                same = (order[i] + sine[i]) % 2 == (order[j] + sine[j]) % 2
                x = (order[i] + sine[i]) % 2
                if not same or (order[i] + order[j] + n + x) % 2:
                    assert abs(J[i, j]) < 1e-9, (n, i, j)
