"""M2L in the order by siblings (131,072 targets and more, that is six levels
and more, which the waves take from a queue per XCD) on sparse leaves, some of
them empty, at orders that the stored values of large clouds do not cover: the
lowest, the highest of one pair per lane, and one whose table of J^T is read
transposed.  The binary64 far field at sampled leaves against the oracle, the
mixed one against it over all points (its bound is one on the norm: a field that
nearly cancels at a single point is further off there)."""
import numpy as np
import pytest

from paper_2002_04894_amd import workloads as W

from test_gpu_parity import F, FP64_TOL, dev, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu

N, L, THETA = 200_000, 6, 0.85
MIXED_TOL = 1e-6


@pytest.fixture(scope="module")
def trees(torch, F, orc):
    x, y, z, q = W.gaussian_mixture(N, seed=9)
    full = np.flatnonzero(np.diff(orc.Tree(x, y, z, L, THETA, leaves=[0]).start(L)))
    assert full.size < 8 ** L  # empty leaves
    leaves = full[[0, full.size // 3, 2 * full.size // 3, -1]]
    ot = orc.Tree(x, y, z, L, THETA, leaves=leaves)
    s, perm = ot.start(L), ot.perm()
    pts = np.concatenate([perm[s[b]:s[b + 1]] for b in leaves])
    gt = F.fmm_build(*(dev(torch, a) for a in (x, y, z)), L, THETA)
    yield ot, gt, q, leaves, pts
    gt.free()


@pytest.mark.parametrize("p,precisions", [(3, (0, 1)), (5, (0, 1)), (14, (0, 1)), (19, (0,))])
def test_far_field_of_sparse_leaves(torch, F, trees, p, precisions):
    ot, gt, q, leaves, pts = trees
    say(f"[siblings] {N} points, {L} levels, order {p}")
    ref = [r[pts] for r in ot.evaluate(q, p, parts=2, leaves=leaves)]
    qd = dev(torch, q)
    outs = [torch.empty_like(qd) for _ in range(4)]
    for prec in precisions:
        say(f"[siblings] precision {prec}")
        F.fmm_evaluate_tree(gt, qd, p, *outs, parts=F.FMM_PART_FAR, precision=prec)
        got = [o.cpu().numpy() for o in outs]
        if prec == 0:
            f64 = got
            for g, r in zip(got, ref):
                assert np.linalg.norm(g[pts] - r) <= FP64_TOL * np.linalg.norm(r)
        else:
            for g, r in zip(got, f64):
                assert np.linalg.norm(g - r) <= MIXED_TOL * np.linalg.norm(r)
