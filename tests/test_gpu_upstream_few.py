"""The upstream chain of few particles with long lists, whose pairs several waves
share, 64 at a time in turn: from one particle on, lists of whole and broken
multiples of 64 pairs, more waves than passes and fewer.  The upstream particle
of every pair equals the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from tests import gpu_common as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_gas,n_src", [(1, 500), (2, 64), (3, 65), (40, 3000), (130, 1001), (300, 640), (2100, 520)])
def test_few_particles(n_gas, n_src):
    import paper_1005_5312_amd as S

    rng = np.random.default_rng(n_gas)
    gas, nhi = rng.random((3, n_gas)), rng.uniform(0.0, 2e-3, n_gas)
    h = np.full(n_gas, 0.5 * (3.0 * 32 / (4.0 * np.pi * max(n_gas, 8))) ** (1.0 / 3.0))
    src, lum = rng.random((3, n_src)), 10.0 ** rng.uniform(47.0, 50.0, n_src)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    sigma = 6.3e-18
    with S.Context(0) as ctx:
        tree, grid = ctx.build_scene(S.Box((0.0, 0.0, 0.0), 1.0, H.KPC), dev(src), dev(lum), dev(gas), dev(h), dev(nhi),
                                     3)
        gam, offs, par, roots = ctx.compute_rates_upstream(tree, grid, gas, h, nhi, None, 0.0, sigma, structure=True)
        gam = gam.cpu().numpy()
        tree.free()
        grid.free()
    box = O.make_box(np.zeros(3), 1.0, H.KPC)
    want, ooffs, opar, ost = O.upstream_rates(O.Tree(box, src, lum), 3, O.grid(box, gas, h, nhi, 3), gas, h, nhi, None,
                                              0.0, sigma, structure=True)
    assert np.array_equal(offs, ooffs) and np.array_equal(par, opar) and roots == int(ost[:, 1].sum())
    rel, ab, _ = H.rel_errors(gam, want)
    assert rel <= H.TOL_FP64 and ab <= H.ABS_FLOOR
