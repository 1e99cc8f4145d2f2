"""The memory a tree keeps."""
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
