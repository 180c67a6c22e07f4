"""P2P of leaves whose targets take several passes, shared by the blocks of one
segment: one leaf, few leaves, cells off the median and separate targets, with
counts at the edges of a pass, in both near-field precisions.  The oracle's near
field to the tolerances of the other parity tests (binary64: 1e-12; binary32:
the bound of the mixed tests' near field).
"""
import numpy as np
import pytest

from test_gpu_mixed import gpu_eval_prec
from test_gpu_parity import F, assert_close, dev, gpu_tree, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels", [(256, 0), (257, 0), (1_500, 0), (8 * 320, 1), (8 * 128 + 1, 1)])
def test_even_leaves(torch, F, orc, n, levels):
    say(f"[p2p] {n}, {levels} levels")
    x, y, z, q = make("uniform", n, seed=31)
    ref = orc.Tree(x, y, z, levels, 0.5).evaluate(q, 4, parts=1)
    gt = gpu_tree(torch, F, x, y, z, levels, 0.5)
    assert_close(gpu_eval_prec(torch, F, gt, q, 4, 1, F.FMM_PREC_F64), ref, what="binary64")
    assert_close(gpu_eval_prec(torch, F, gt, q, 4, 1, F.FMM_PREC_F32), ref, tol=1e-4, what="binary32")
    gt.free()


@pytest.mark.parametrize("n,m,levels", [(4_000, 0, 2), (3_000, 5_000, 1), (2_000, 700, 0)])
def test_targets_equal_the_direct_sum(torch, F, n, m, levels):
    """Targets among sources, cells off the median, theta = 0: every pair is
    near, so the result is the direct sum (1e-12, summation order only)."""
    say(f"[p2p] {n} + {m}, {levels} levels, eta 0.2")
    x, y, z, q = make("uniform", n, seed=32)
    X = [dev(torch, a) for a in (x, y, z)]
    T = [np.ascontiguousarray(a) for a in make("plummer", m or n, seed=33)[:3]]
    tree = F.fmm_build_ex(*X, levels, 0.0, eta=0.2, targets=[dev(torch, a) for a in T])
    outs = [torch.empty(len(T[0]), dtype=torch.float64, device="cuda") for _ in range(4)]
    F.fmm_evaluate_targets(tree, dev(torch, q), 3, *outs, precision=F.FMM_PREC_F64)
    torch.cuda.synchronize()
    d = [t[:, None] - s[None, :] for t, s in zip(T, (x, y, z))]
    inv = 1.0 / np.sqrt(d[0] ** 2 + d[1] ** 2 + d[2] ** 2)
    ref = [(q * inv).sum(1)] + [(q * inv ** 3 * c).sum(1) for c in d]
    for u, v in zip(outs, ref):
        assert np.linalg.norm(u.cpu().numpy() - v) <= 1e-12 * np.linalg.norm(v)
    tree.free()
