"""Trees with planes off the median whose bisection rounds run chunked on
unequal segments: bit for bit the oracle's.  That at least two such rounds meet
the condition of the chunked kernels (no segment below 8,192 points, the largest
of 32,768 or more, in this round and all before) is read off the oracle's
segments."""
import numpy as np
import pytest

from paper_2002_04894_amd import workloads as W

from test_gpu_f4 import gpu_build
from test_gpu_parity import F, assert_tree_equal, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def segments(ot, depth):
    """points of the 2^depth segments of a bisection round"""
    n = np.diff(ot.start(-(-depth // 3)))
    return n.reshape(2 ** depth, -1).sum(axis=1)


@pytest.mark.parametrize("gen,n,eta", [
    ("gaussian_mixture", 240_000, 0.3), ("gaussian_mixture", 120_000, 0.3), ("spherical_gaussian", 400_000, 0.0),
    ("helix", 200_000, 0.8), ("plummer", 300_000, 0.5),
])
def test_unequal_chunked_rounds(torch, F, orc, gen, n, eta):
    say(f"[eta] chunked {gen} {n}, eta {eta}")
    x, y, z, _ = getattr(W, gen)(n, seed=9)
    ot = orc.Tree(x, y, z, 2, 0.5, eta=eta)
    chunked = 0
    for depth in range(1, 6):
        s = segments(ot, depth)
        if s.min() < 8_192 or s.max() < 32_768:
            break
        chunked += s.min() != s.max()
    assert chunked >= 2
    gt = gpu_build(torch, F, x, y, z, 2, 0.5, eta)
    assert_tree_equal(F, gt, ot, 2)
    gt.free()
