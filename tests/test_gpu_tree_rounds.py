"""Tree and lists bit for bit against the oracle at the sizes where a bisection
round or a scan changes its kernels: one block of 64, 256 or 1,024 threads per
segment, the chunked rounds (segments of 32,768 points and more), levels with
more than 8,192 boxes, and with half-way planes (eta 0.5), whose segments are
unequal.
"""
import pytest

from test_gpu_f4 import gpu_build
from test_gpu_parity import F, assert_tree_equal, gpu_tree, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gen,n,levels", [
    ("uniform", 128, 1), ("uniform", 129, 1), ("gmix", 2048, 1), ("gmix", 2049, 1), ("plummer", 32_767, 2),
    ("plummer", 32_768, 2), ("gmix", 65_535, 2), ("uniform", 65_537, 2), ("quantized", 70_001, 2),
    ("uniform", 40_000, 5),
])
def test_median_rounds(torch, F, orc, gen, n, levels):
    say(f"[tree] {gen} {n}, {levels} levels")
    x, y, z, _ = make(gen, n, seed=31)
    theta = 0.9 if levels == 5 else 0.5
    gt = gpu_tree(torch, F, x, y, z, levels, theta)
    assert_tree_equal(F, gt, orc.Tree(x, y, z, levels, theta), levels)
    gt.free()


@pytest.mark.parametrize("gen,n", [("gmix", 1_025), ("plummer", 33_000), ("uniform", 80_000)])
def test_half_way_rounds(torch, F, orc, gen, n):
    say(f"[tree] {gen} {n}, eta 0.5")
    x, y, z, _ = make(gen, n, seed=32)
    gt = gpu_build(torch, F, x, y, z, 2, 0.5, 0.5)
    assert_tree_equal(F, gt, orc.Tree(x, y, z, 2, 0.5, eta=0.5), 2)
    gt.free()
