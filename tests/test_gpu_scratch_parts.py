"""Scratch of an evaluation by what is asked for: the near field alone takes
none of the far field's buffers, the far field alone none of the near field's
partial sums, an evaluation at the sources nothing for the separate targets;
so the entry point that allocates nothing runs parts whose sum it refuses."""
import numpy as np
import pytest

from paper_2002_04894_amd import workloads as W

from test_gpu_boundary import Counting
from test_gpu_parity import F, dev, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu

ARRAY = 64 << 20  # bytes of the fixed array


def test_noalloc_parts_that_fit(torch, F):
    # 8 leaves of 28,331 points: eight segments each, so 256 bytes of partial
    # sums per point beside 8 of charges and 32 of far field; the expansions of
    # the 9 boxes at order 20 no longer fit beside all of them
    n, p = 226_650, 20
    assert 296 * n <= ARRAY - 12 * 256 < 296 * n + 9 * 441 * 8
    say(f"[noalloc] parts of {n} points, 1 level, p {p}")
    d = [dev(torch, a) for a in W.uniform_cube(n, seed=1)]
    t = F.fmm_build(*d[:3], 1, 0.5)
    for parts in (F.FMM_PART_NEAR, F.FMM_PART_FAR):
        ref, out = ([torch.empty_like(d[3]) for _ in range(4)] for _ in range(2))
        F.fmm_evaluate_tree(t, d[3], p, *ref, parts=parts)
        F.fmm_evaluate_tree_noalloc(t, d[3], p, *out, parts=parts)
        torch.cuda.synchronize()
        for u, v in zip(out, ref):
            assert torch.equal(u, v)
    with pytest.raises(F.FMMError) as e:
        F.fmm_evaluate_tree_noalloc(t, d[3], p, *out)
    assert e.value.code == F.FMM_EINVAL and "scratch" in str(e.value)
    t.free()


def test_scratch_of_parts_and_of_trees_with_targets(torch, F):
    n, m, L, p = 20_000, 200_000, 3, 15
    nbox = (8 ** (L + 1) - 1) // 7
    x, y, z, q = W.uniform_cube(n, seed=2)
    d = [dev(torch, a) for a in (x, y, z, q)]
    lo, hi = [a.min() for a in (x, y, z)], [a.max() for a in (x, y, z)]
    r = np.random.default_rng(3).random((3, m))
    T = tuple(dev(torch, l + (h - l) * (0.1 + 0.8 * c)) for l, h, c in zip(lo, hi, r))
    plain, targets = F.fmm_build(*d[:3], L, 0.5), F.fmm_build_ex(*d[:3], L, 0.5, targets=T)
    scratch = F.fmm_tree_bytes(plain, p)[1]
    outs = [torch.empty_like(d[3]) for _ in range(4)]
    c = Counting(torch)
    F.fmm_set_allocator(c.alloc, c.free)
    try:
        def peak(tree, parts):
            c.peak = 0
            F.fmm_evaluate_tree(tree, d[3], p, *outs, parts=parts)
            torch.cuda.synchronize()
            assert c.bytes() == 0
            return c.peak
        assert peak(plain, F.FMM_PART_ALL) == scratch
        # less by the multipoles and the far field at least
        assert peak(plain, F.FMM_PART_NEAR) <= scratch - nbox * (p + 1) ** 2 * 8 - 32 * n
        assert peak(targets, F.FMM_PART_ALL) == scratch
    finally:
        F.fmm_set_allocator()
    plain.free()
    targets.free()
