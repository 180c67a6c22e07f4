"""Clouds and targets with a coordinate that is not acceptable (NaN, infinite,
beyond 1e300) are refused, whatever the bisection rounds meet before the host
looks at the flag: segments of two points of which one is not acceptable,
rounds of one block and chunked ones, planes off the median.  The build after
a refused one is the oracle's."""
import numpy as np
import pytest

from paper_2002_04894_amd import workloads as W

from test_gpu_parity import assert_tree_equal, dev, torch, F  # noqa: F401

pytestmark = pytest.mark.gpu

VALUES = [np.nan, -np.nan, np.inf, -np.inf, 2e300]


@pytest.mark.parametrize("eta", [1.0, 0.5])
@pytest.mark.parametrize("n,L,nbad", [(2, 1, 1), (64, 2, 1), (70, 2, 3), (1000, 3, 400), (40_000, 3, 1), (70_000, 2, 70_000)])
def test_unacceptable_coordinates_refused(torch, F, orc, n, L, nbad, eta):
    rng = np.random.default_rng(n + L)
    good = W.uniform_cube(n, seed=n)[:3]
    for k, v in enumerate(VALUES):
        for targets in (False, True):
            print(f"[nonfinite] n={n} L={L} nbad={nbad} eta={eta} value={v} targets={targets}", flush=True)
            pts = [a.copy() for a in good]
            for i in rng.permutation(n)[:nbad]:
                pts[(i + k) % 3][i] = v
            with pytest.raises(F.FMMError) as e:
                if targets:
                    F.fmm_build_ex(*(dev(torch, a) for a in good), L, 0.5, eta, targets=tuple(dev(torch, a) for a in pts))
                else:
                    F.fmm_build_ex(*(dev(torch, a) for a in pts), L, 0.5, eta)
            assert e.value.code == F.FMM_EINVAL
    ot = orc.Tree(*good, L, 0.5, eta=eta)
    gt = F.fmm_build_ex(*(dev(torch, a) for a in good), L, 0.5, eta)
    assert_tree_equal(F, gt, ot, L)
    gt.free()
