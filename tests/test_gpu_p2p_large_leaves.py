"""Near field of leaves so large that a segment (about 8,192 sources) has one,
two or a few entries: the waves that share it change with that number.  Against
the direct sum (one leaf: nothing but the near field)."""
import numpy as np
import pytest

from paper_2002_04894_amd import workloads as W

from test_gpu_parity import F, FP64_TOL, dev, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


# points per leaf: 500, 1,500, 2,500, 4,000, 8,750 in 8 leaves
@pytest.mark.parametrize("n", [4_000, 12_000, 20_003, 32_000, 70_001])
def test_large_leaves(torch, F, orc, n):
    say(f"[p2p] {n} points, 8 leaves")
    x, y, z, q = W.gaussian_mixture(n, seed=41)
    d = [dev(torch, a) for a in (x, y, z, q)]
    outs = [torch.empty_like(d[0]) for _ in range(4)]
    t = F.fmm_build(*d[:3], 1, 0.5)
    F.fmm_evaluate_tree(t, d[3], 0, *outs, parts=F.FMM_PART_NEAR)
    got = [o.cpu().numpy() for o in outs]
    t.free()
    some = np.random.default_rng(n).integers(0, n, 200)
    ot = orc.Tree(x, y, z, 0, 0.5, targets=(x[some], y[some], z[some]))
    ref = ot.evaluate_targets(q, 0)
    # all eight leaves are strongly connected at theta 0.5: the near field is the whole sum
    for g, r in zip(got, ref):
        assert np.linalg.norm(g[some] - r) <= FP64_TOL * np.linalg.norm(r)
