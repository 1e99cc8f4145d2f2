"""Gas grids with kernels that reach over many cells: a class of at most as many
particles as its stencil has rows is taken whole, a larger one row by row; and
the price of a few wide kernels among many narrow ones."""
from __future__ import annotations

import time

import numpy as np
import pytest

from oracle import oracle as O
from tests import gpu_common as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# 16^3 cells and h = 0.1: a reach of 3.2 cells, pi 3.7^2 = 43.0 rows
@pytest.mark.parametrize("n,wide,h_wide,log2", [(43, 0, 0.0, 4), (44, 0, 0.0, 4), (9, 0, 0.0, 1), (5, 0, 0.0, 1),
                                                (700, 1, 3.0, 3), (2000, 7, 0.4, 4), (2000, 300, 0.4, 4),
                                                (900, 17, 0.3, 5), (4000, 1, 0.7, 6), (500, 400, 0.2, 6),
                                                (300, 9, 0.5, 7)])
def test_values(n, wide, h_wide, log2):
    import paper_1005_5312_amd as S

    rng = np.random.default_rng(n + wide + log2)
    xyz, nhi = rng.random((3, n)), rng.uniform(0.0, 1e-2, n)
    h = np.full(n, 0.1 if wide == 0 else 0.04)
    h[rng.permutation(n)[:wide]] = h_wide
    with S.Context(0) as ctx:
        grid = ctx.build_gas_grid(S.Box((0.0, 0.0, 0.0), 1.0, H.KPC), _dev(xyz), _dev(h), _dev(nhi), log2)
        got = ctx.grid_export(grid)
        grid.free()
    want = O.grid(O.make_box(np.zeros(3), 1.0, H.KPC), xyz, h, nhi, log2).reshape(got.shape)
    # sums of at most n positive terms, each a kernel weight good to ~1e-15 of
    # the kernel's scale; only weights at the support's edge lose relative digits
    assert np.array_equal(got == 0.0, want == 0.0)
    scale = np.where(want > 0.0, want, 1.0)
    assert np.max(np.abs(got - want) / scale) <= 1e-12 + 4e-16 * n


def test_one_wide_kernel_costs_little():
    """One kernel wider than the box adds a test per centre, not a look-up of
    every row: the build takes about as long as without it (8 times as long by
    rows; 4 allows for a slow first call of either)."""
    import paper_1005_5312_amd as S

    n = 1 << 18
    rng = np.random.default_rng(5)
    xyz, nhi = _dev(rng.random((3, n))), _dev(np.full(n, 1e-3))
    h = np.full(n, 0.5 * (3.0 * 32 / (4.0 * np.pi * n)) ** (1.0 / 3.0))
    took = []
    with S.Context(0) as ctx:
        for first in (h[0], 0.6):
            h[0] = first
            hd, best = _dev(h), np.inf
            for _ in range(6):
                ctx.synchronize()
                t = time.perf_counter()
                ctx.build_gas_grid(S.Box((0.0, 0.0, 0.0), 1.0, H.KPC), xyz, hd, nhi, 6).free()
                best = min(best, time.perf_counter() - t)
            took.append(best)
    assert took[1] <= 4.0 * took[0], took
