"""Trees with more cells above 128 sources at one level than the block that sums
them has threads, and with many such levels; and the memory a tree keeps."""
from __future__ import annotations

import numpy as np
import pytest

from tests import gpu_common as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _tree(ctx, xyz, lum):
    import paper_1005_5312_amd as S

    return ctx.build_source_tree(S.Box((0.0, 0.0, 0.0), 1.0, H.KPC), torch.from_numpy(xyz).cuda(),
                                 torch.from_numpy(lum).cuda())


@pytest.mark.parametrize("kind,n", [("uniform", 1 << 20), ("nested", 400000), ("points", 300000)])
def test_moments(kind, n):
    import paper_1005_5312_amd as S

    rng = np.random.default_rng(n)
    xyz = rng.random((3, n))
    if kind == "nested":          # large cells down to the last levels
        xyz = 0.3 + xyz * 2.0 ** -rng.integers(0, 20, n)[None, :] * 0.5
    elif kind == "points":        # 1500 points of 200 sources: large level-21 cells
        xyz = rng.random((3, 1500))[:, rng.integers(0, 1500, n)]
    xyz, lum = np.ascontiguousarray(xyz), 10.0 ** rng.uniform(47.0, 50.0, n)
    with S.Context(0) as ctx:
        tree = _tree(ctx, xyz, lum)
        e = ctx.tree_export(tree)
        tree.free()
    _, first, count, _ = e["link"].T
    level = e["geo"][:, 3] & 0xFF
    L, X = lum[e["perm"]], xyz[:, e["perm"]]
    for lv in np.unique(level):
        p = np.flatnonzero((level == lv) & (count > 1))    # disjoint runs of sources
        if p.size == 0:
            continue
        ends = np.stack([first[p], first[p] + count[p]], axis=1).ravel()
        runs = lambda v: np.add.reduceat(np.append(v, 0.0), ends)[::2]  # noqa: E731
        tot = runs(L)
        # sums of at most n positive terms: relative error at most n ulp on each side
        tol = 4e-16 * count[p]
        assert np.all(np.abs(e["mom"][p, 3] - tot) <= tol * tot), lv
        for k in range(3):
            assert np.all(np.abs(e["mom"][p, k] - runs(X[k] * L) / tot) <= 3.0 * tol + 1e-15), lv


def test_bytes_per_source():
    """60 bytes a source, and 128 for each of at most two nodes."""
    import paper_1005_5312_amd as S

    n = 100000
    rng = np.random.default_rng(1)
    with S.Context(0) as ctx:
        before = ctx.bytes_in_use()
        tree = _tree(ctx, rng.random((3, n)), np.ones(n))
        kept = ctx.bytes_in_use() - before
        tree.free()
        assert ctx.bytes_in_use() == before
    assert kept <= 316 * n + 16 * 256, kept / n
