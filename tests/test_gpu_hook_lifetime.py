"""A tree built with an allocator hook is freed through it, also after the hook
has been replaced and nothing else holds its callables."""
import gc
import weakref

import pytest

from paper_2002_04894_amd import workloads as W

from test_gpu_boundary import Counting
from test_gpu_parity import F, dev, say, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def test_tree_outlives_its_hook(torch, F):
    say("[hook] freed after the hook was replaced")
    c = Counting(torch)
    free = lambda p, s: c.free(p, s)  # noqa: E731
    hook = weakref.ref(free)
    F.fmm_set_allocator(c.alloc, free)
    del free
    try:
        t = F.fmm_build(*(dev(torch, a) for a in W.uniform_cube(3000, seed=1)[:3]), 2, 0.5)
    finally:
        F.fmm_set_allocator()
    gc.collect()
    assert hook() is not None and c.bytes() == F.fmm_tree_bytes(t, 3)[0] > 0
    t.free()
    assert c.bytes() == 0
    del t
    gc.collect()
    assert hook() is None
