"""Near field at the leaf sizes where the split of a wave between targets and
source streams changes (one to four targets per lane, lanes left over, several
passes over one leaf), and with one, four and eight waves per work item,
against the oracle's near field: 1e-12 for binary64 (summation order only),
1e-4 for the binary32 near field, the accuracy it is offered for.
"""
import pytest

from test_gpu_mixed import gpu_eval_prec
from test_gpu_parity import F, assert_close, gpu_tree, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels", [
    (1, 0), (2, 0), (15, 0), (39, 0), (64, 0), (65, 0), (93, 0), (129, 0), (256, 0), (257, 0), (700, 0),  # one leaf
    (8 * 64 * 23, 3),   # 512 leaves of 23: eight waves per item
    (512 * 41 + 77, 3),  # ragged, some leaves one point more
    (20_000, 3),         # a few thousand items at theta 0: four waves
    (9_000, 4),          # 4,096 leaves of two or three points: one wave
])
def test_near_field(torch, F, orc, n, levels):
    say(f"[p2p] n={n} levels={levels}")
    theta = 0.0 if n == 20_000 else 0.6
    x, y, z, q = make("uniform", n, seed=21)
    ref = orc.Tree(x, y, z, levels, theta).evaluate(q, 2, parts=1)
    gt = gpu_tree(torch, F, x, y, z, levels, theta)
    assert_close(gpu_eval_prec(torch, F, gt, q, 2, 1, F.FMM_PREC_F64), ref, what="binary64")
    assert_close(gpu_eval_prec(torch, F, gt, q, 2, 1, F.FMM_PREC_F32), ref, tol=1e-4, what="binary32")
    gt.free()
