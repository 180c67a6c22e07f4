"""M2L over the ways its targets are dealt out: one target per block (up to
three levels), single waves with the long lists shared by blocks (four levels,
skewed lists), at orders on both sides of the two-waves limit, against the
oracle's far field.  Tolerances as for the other parity tests: 1e-12 for
binary64 (summation order only), 1e-6 for the binary32 M2L.  (Trees with
siblings side by side in the order are covered by the stored 2^24- and
2^27-point values.)
"""
import pytest

from paper_2002_04894_amd import workloads as W
from test_gpu_mixed import MIXED_TOL, gpu_eval_prec
from test_gpu_parity import F, assert_close, gpu_tree, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dist,n,levels,theta,p", [
    ("uniform", 300, 2, 0.6, 7),      # 72 targets, eight of them without a list
    ("sphere", 5_000, 3, 0.4, 14),    # 584 targets, lists of very different lengths
    ("plummer", 6_000, 4, 0.55, 6),   # 4,680 targets, no list beyond a wave's share
    ("sphere", 9_000, 4, 0.4, 5),     # the same, some beyond it
    ("sphere", 5_000, 4, 0.5, 16),    # one wave per SIMD
])
def test_far_field(torch, F, orc, dist, n, levels, theta, p):
    say(f"[m2l] {dist} {n}, {levels} levels, theta {theta}, p {p}")
    x, y, z, q = W.sphere_surface(n, seed=11) if dist == "sphere" else make(dist, n, seed=11)
    ref = orc.Tree(x, y, z, levels, theta).evaluate(q, p, parts=2)
    gt = gpu_tree(torch, F, x, y, z, levels, theta)
    assert F.fmm_tree_stats(gt)[0] > 0
    assert_close(gpu_eval_prec(torch, F, gt, q, p, 2, F.FMM_PREC_F64), ref, what="binary64")
    assert_close(gpu_eval_prec(torch, F, gt, q, p, 2, F.FMM_PREC_MIXED), ref, tol=MIXED_TOL, what="mixed")
    gt.free()
