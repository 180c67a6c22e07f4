"""P2M with several waves per leaf (up to 512 leaves; four up to order 12, two
above) and one (more leaves): leaves with fewer points than one wave takes,
more than all waves take at once, and remainders, against the oracle's far
field.  Tolerance as for the other parity tests: 1e-12 (summation order only).
"""
import pytest

from test_gpu_mixed import gpu_eval_prec
from test_gpu_parity import F, assert_close, gpu_tree, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels,theta,p", [
    (64 * 300, 2, 0.6, 3),        # 300 points per leaf: five passes over four waves
    (64 * 257 + 13, 2, 0.6, 12),  # 257 or 258: a wave's second pass of one point
    (64 * 129, 2, 0.6, 13),       # two waves, one point left over
    (64 * 64, 2, 0.6, 20),        # exactly one wave's points
    (100, 2, 0.5, 8),             # one or two points per leaf
    (4_200, 4, 0.6, 5),           # 4,096 leaves, one wave each
])
def test_far_field(torch, F, orc, n, levels, theta, p):
    say(f"[p2m] {n}, {levels} levels, theta {theta}, p {p}")
    x, y, z, q = make("uniform", n, seed=21)
    ref = orc.Tree(x, y, z, levels, theta).evaluate(q, p, parts=2)
    gt = gpu_tree(torch, F, x, y, z, levels, theta)
    assert F.fmm_tree_stats(gt)[0] > 0
    assert_close(gpu_eval_prec(torch, F, gt, q, p, 2, F.FMM_PREC_F64), ref)
    gt.free()
