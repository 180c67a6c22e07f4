"""Builds cut small buffers out of shared blocks and small evaluations run in
one block: over sizes on both sides of the sharing and one-block limits, what
the allocator holds is what the tree states, everything comes back, and the
results equal those of the entry point that allocates nothing, bitwise.
"""
import numpy as np
import pytest

from test_gpu_boundary import Counting
from test_gpu_parity import F, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,levels,p,prec", [
    (1, 0, 0, 3, 0),          # the smallest buffers
    (700, 0, 0, 3, 1),        # no expansions
    (1_000, 5_000, 2, 9, 0),  # separate targets
    (9_000, 0, 3, 15, 0),     # more than one shared block
    (120_000, 0, 4, 6, 1),    # evaluation in one block
    (300_000, 0, 4, 6, 1),    # coordinates in blocks of their own
])
def test_blocks(torch, F, n, m, levels, p, prec):
    say(f"[blocks] {n} + {m}, {levels} levels, p {p}, precision {prec}")
    x, y, z, q = make("uniform", n, seed=3)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    X, qd = [dev(a) for a in (x, y, z)], dev(q)
    T = [dev(a) for a in make("uniform", m, seed=4)[:3]] if m else None
    c = Counting(torch)
    F.fmm_set_allocator(c.alloc, c.free)
    try:
        tree = F.fmm_build_ex(*X, levels, 0.5, targets=T) if m else F.fmm_build(*X, levels, 0.5)
        torch.cuda.synchronize()
        own, scratch = F.fmm_tree_bytes(tree, p, prec)
        assert c.bytes() == own
        c.peak = own
        outs = [torch.empty_like(qd) for _ in range(4)]
        F.fmm_evaluate_tree(tree, qd, p, *outs, precision=prec)
        if m:
            touts = [torch.empty(m, dtype=torch.float64, device="cuda") for _ in range(4)]
            F.fmm_evaluate_targets(tree, qd, p, *touts, precision=prec)
        torch.cuda.synchronize()
        assert c.bytes() == own and c.peak - own <= scratch
        ref = [torch.empty_like(qd) for _ in range(4)]
        F.fmm_evaluate_tree_noalloc(tree, qd, p, *ref, precision=prec)
        torch.cuda.synchronize()
        for u, v in zip(outs, ref):
            assert torch.equal(u, v)
        tree.free()
        assert c.bytes() == 0
    finally:
        F.fmm_set_allocator()
