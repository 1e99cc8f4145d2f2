"""FP32C rates and the order in which their terms are summed: the equilibrium
loops sum them depth first, the other calls frame by frame.  The two are bounded
against each other, and both walks against the oracle on trees whose sources are
far apart (test_gpu_sibling_walk compares tile sizes, which all take one walk)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from tests import gpu_common as H
from tests.test_gpu_sibling_walk import _sources

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIGMA = 6.3e-18


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("kind", ["one", "bucket", "deep", "lattice"])
@pytest.mark.parametrize("theta", [0.3, 1.0])
def test_loop_against_plain_call(kind, theta):
    """The same terms, each sum with Kahan compensation: 2 units of 2^-24 from the
    exact sum, and half an FP32 ulp more when stored, on either side."""
    import paper_1005_5312_amd as S

    rng = np.random.default_rng(14)
    src, lum = _sources(kind, rng)
    n = 5000
    gas, h = _dev(rng.random((3, n))), _dev(np.full(n, 0.1))
    nh, x0 = _dev(rng.uniform(0.5e-3, 2e-3, n)), _dev(rng.uniform(0.1, 1.0, n))
    box = S.Box((0.0, 0.0, 0.0), 1.0, H.KPC)
    with S.Context(0) as ctx:
        tree = ctx.build_source_tree(box, _dev(src), _dev(lum))
        _, loop, _, _ = ctx.ionization_equilibrium(tree, gas, h, nh, x0, 4, theta, SIGMA, 2.59e-13, "fp32c", max_iter=1,
                                                   tol=0.0)
        grid = ctx.build_gas_grid(box, gas, h, nh * x0, 4)
        plain = ctx.compute_rates(tree, grid, gas, None, theta, SIGMA, "fp32c")
        ctx.synchronize()
        grid.free()
        tree.free()
    a, b = loop.double().cpu().numpy(), plain.double().cpu().numpy()
    assert np.isfinite(a).all() and a.max() > 0
    assert np.max(np.abs(a - b) / np.maximum(b, 1e-300)) <= 2 * (2.0 * 2.0 ** -24 + 2.0 ** -24) * (1 + 1e-3)


@pytest.mark.parametrize("kind", ["one", "lattice"])
@pytest.mark.parametrize("theta", [0.0, 0.7, 1.0])
@pytest.mark.parametrize("loop", [False, True])
def test_against_oracle(kind, theta, loop):
    import paper_1005_5312_amd as S

    rng = np.random.default_rng(15)
    src, lum = _sources(kind, rng)
    n = 700
    gas, h, nhi = rng.random((3, n)), np.full(n, 0.12), rng.uniform(0.0, 2e-3, n)
    box, obox = S.Box((0.0, 0.0, 0.0), 1.0, H.KPC), O.make_box(np.zeros(3), 1.0, H.KPC)
    want = O.rates(O.Tree(obox, src, lum), 4, O.grid(obox, gas, h, nhi, 4), gas, np.full(n, -1, np.int64), theta, SIGMA)
    with S.Context(0) as ctx:
        tree, grid = ctx.build_scene(box, _dev(src), _dev(lum), _dev(gas), _dev(h), _dev(nhi), 4)
        for tile in (1, 8, 16, 32, 64):
            ctx.set_tile_targets(tile)
            if loop:
                got = ctx.ionization_equilibrium(tree, _dev(gas), _dev(h), _dev(nhi), _dev(np.ones(n)), 4, theta, SIGMA,
                                                 2.59e-13, "fp32c", max_iter=1, tol=0.0)[1]
            else:
                got = ctx.compute_rates(tree, grid, _dev(gas), None, theta, SIGMA, "fp32c")
            ctx.synchronize()
            rel, ab, _ = H.rel_errors(got.double().cpu().numpy(), want)
            assert rel <= H.TOL_FP32C and ab <= H.ABS_FLOOR, tile
        tree.free()
        grid.free()
