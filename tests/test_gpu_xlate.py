"""M2M, L2L and the leaf operators at the high orders, on both sides of the
order from which the translations leave the matrix cores, and for boxes whose
children share their centre (a translation by zero), against the oracle's far
field.  Tolerance as for the other parity tests: 1e-12 (summation order only).
"""
import numpy as np
import pytest

from paper_2002_04894_amd import workloads as W
from test_gpu_mixed import gpu_eval_prec
from test_gpu_parity import F, assert_close, gpu_tree, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def clusters(n):
    """n points at eight places: below level 1 every box is a point."""
    x, y, z, q = make("uniform", n, seed=5)
    k = np.arange(n) % 8
    return (k & 1) * 1.0, (k >> 1 & 1) * 1.0, (k >> 2) * 1.0, q


@pytest.mark.parametrize("dist,n,levels,theta,p", [
    ("uniform", 1_500, 2, 0.6, 14),
    ("sphere", 3_000, 3, 0.5, 15),
    ("sphere", 1_500, 3, 0.5, 17),
    ("clusters", 512, 3, 0.5, 18),
    ("uniform", 1_500, 3, 0.5, 18),
    ("uniform", 1_500, 3, 0.5, 19),
    ("uniform", 1_500, 3, 0.5, 1),
])
def test_far_field(torch, F, orc, dist, n, levels, theta, p):
    say(f"[xlate] {dist} {n}, {levels} levels, theta {theta}, p {p}")
    if dist == "clusters":
        x, y, z, q = clusters(n)
    else:
        x, y, z, q = W.sphere_surface(n, seed=12) if dist == "sphere" else make(dist, n, seed=12)
    ref = orc.Tree(x, y, z, levels, theta).evaluate(q, p, parts=2)
    gt = gpu_tree(torch, F, x, y, z, levels, theta)
    assert F.fmm_tree_stats(gt)[0] > 0
    assert_close(gpu_eval_prec(torch, F, gt, q, p, 2, F.FMM_PREC_F64), ref)
    gt.free()
