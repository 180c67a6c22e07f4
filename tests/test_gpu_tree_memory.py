"""What a kept tree holds beside its arrays: at most about as much again, where
its build held the points twice (few boxes for the points, planes off the
median)."""
import numpy as np
import pytest

from test_gpu_boundary import Counting
from test_gpu_parity import F, dev, make, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def arrays(F, t, n, m, L):
    """bytes of the tree's arrays (the near field's plan aside: 12 bytes per
    segment of about 8,192 sources)"""
    b = 28 * n + (32 * m + 4 * (8 ** L + 1) + 8 * (8 ** L + 1) if m else 0)
    for l in range(L + 1):
        nb = 8 ** l
        b += 80 * nb + 4 * (nb + 1) + 2 * 8 * (nb + 1) + 4 * sum(F.fmm_tree_lists(t, l, k)[0][-1] for k in (0, 1))
    return b + 4 * (8 ** (L + 1) - 1) // 7 + 2 * 8 * (8 ** L + 1)


@pytest.mark.parametrize("n,m,L,eta", [
    (100, 0, 0, 1.0), (1_000, 0, 2, 1.0), (4_000, 0, 2, 1.0), (10_000, 0, 3, 1.0), (30_000, 0, 3, 1.0),
    (60_000, 0, 3, 1.0), (60_000, 50_000, 3, 0.5), (100_000, 0, 3, 0.3), (130_000, 0, 4, 1.0),
    (226_650, 0, 1, 1.0), (300_000, 0, 4, 1.0),
])
def test_kept_tree_and_its_arrays(torch, F, n, m, L, eta):
    d = [dev(torch, a) for a in make("gmix", n, seed=51)[:3]]
    T = tuple(dev(torch, a) for a in make("gmix", m, seed=52)[:3]) if m else None
    c = Counting(torch)
    F.fmm_set_allocator(c.alloc, c.free)
    try:
        t = F.fmm_build_ex(*d, L, 0.5, eta, targets=T)
        own, least = F.fmm_tree_bytes(t, 3)[0], arrays(F, t, n, m, L)
        say(f"[memory] {n} + {m} points, {L} levels, eta {eta}: {own} bytes, arrays {least}, {c.calls} allocations")
        held = c.bytes()
        t.free()
        assert held == own and c.bytes() == 0
        assert least <= own <= 2.1 * least + (64 << 10)
    finally:
        F.fmm_set_allocator()
