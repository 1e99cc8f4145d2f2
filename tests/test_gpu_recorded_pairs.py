"""When the equilibrium loops record the grid's (cell, particle) pairs: not in a
loop that ends in its first iteration; and the same results with and without."""
from __future__ import annotations

import numpy as np
import pytest

from tests import gpu_common as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _loop(ctx, xyz, h, log2, **kw):
    import paper_1005_5312_amd as S

    n = h.numel()
    tree = ctx.build_source_tree(S.Box((0.0, 0.0, 0.0), 1.0, H.KPC * 13.2), _dev(np.full((3, 1), 0.5)),
                                 _dev(np.array([5e48])))
    nh, x0 = torch.full_like(h, 1e-3), torch.full_like(h, 0.999)
    out = ctx.ionization_equilibrium(tree, xyz, h, nh, x0, log2, prec="fp64", **kw)
    tree.free()
    return out


def test_one_iteration_holds_no_pairs():
    """2^18 particles on 64^3 cells have about 32 pairs a cell, at least 100 MB
    recorded; the rest of the loop's memory is about 60 MB."""
    import paper_1005_5312_amd as S

    n = 1 << 18
    xyz = _dev(np.random.default_rng(3).random((3, n)))
    h = torch.full((n,), 0.5 * (3.0 * 32 / (4.0 * np.pi * n)) ** (1.0 / 3.0), dtype=torch.float64, device="cuda")
    taken = {}
    for tol, iterations in ((2.0, 1), (0.0, 2)):
        with S.Context(0) as ctx:
            torch.cuda.synchronize()
            before = torch.cuda.mem_get_info()[0]
            _, _, done, _ = _loop(ctx, xyz, h, 6, max_iter=2, tol=tol)
            taken[done] = before - torch.cuda.mem_get_info()[0]
            assert done == iterations
    assert taken[2] - taken[1] >= 90e6, taken


@pytest.mark.parametrize("crowd", [0, 2039, 2056, 6000])
@pytest.mark.parametrize("graphs", [True, False])
def test_values_with_and_without_pairs(crowd, graphs):
    """Also crowds of up to 255 particles a slice and of more, which are not recorded."""
    import paper_1005_5312_amd as S

    n = 9000
    rng = np.random.default_rng(crowd)
    xyz = rng.random((3, n))
    xyz[:, :crowd] = 0.52 + 0.01 * xyz[:, :crowd]
    xyz, h = _dev(xyz), _dev(np.full(n, 0.07))
    got = {}
    with S.Context(0) as ctx:
        ctx.set_graph_replay(graphs)
        for pairs in (True, False):
            ctx.set_grid_pairs(pairs)
            for k in (1, 2, 3, 5):
                got[pairs, k] = _loop(ctx, xyz, h, 4, max_iter=k, tol=0.0)
    for k in (1, 2, 3, 5):
        a, b = got[True, k], got[False, k]
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2:] == b[2:], k
