"""Targets per wave (csrc/tiles.h), compiled on their own with the host compiler:
the choice on both sides of its lines, and the autotuner's size classes, which
must tell apart whatever the choice depends on."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1005_5312_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "tiles.h"
int main(int argc, char **argv)
{
    start::BatchSize b;
    b.total = atoll(argv[1]), b.max_t = atoll(argv[2]), b.max_src = atoll(argv[3]);
    b.theta = atof(argv[4]), b.fp64 = atoi(argv[5]) != 0, b.grid = atoi(argv[6]);
    printf("%d", start::tile_from_size(b));
    for (int v : start::tile_class(b)) printf(" %d", v);
    printf("\n");
    return 0;
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "t.cpp").write_text(PROGRAM)
    try:
        subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True,
                       capture_output=True, text=True)
    except FileNotFoundError:
        pytest.skip("no host C++ compiler")

    def run(n, n_src, theta=1.0, prec="fp32c", max_t=None, grid=128):
        args = map(str, (n, max_t or n, n_src, theta, int(prec == "fp64"), grid))
        out = subprocess.run([str(d / "t"), *args], check=True, capture_output=True, text=True).stdout.split()
        return int(out[0]), tuple(map(int, out[1:]))
    return run


ALL = 0   # every particle a source
K = 1 << 16


@pytest.mark.parametrize("n,n_src,theta,prec,tile", [
    # small calls: about n / 4096
    (1000, ALL, 1.0, "fp32c", 1), (8192, ALL, 1.0, "fp32c", 2), (16457, ALL, 1.0, "fp32c", 4), (2 * K, ALL, 1.0, "fp64", 8),
    # every particle a source: 16 up to 7 * 2^16 in FP32C, to 2^18 in FP64
    (4 * K, ALL, 1.0, "fp32c", 16), (330001, ALL, 1.0, "fp32c", 16), (370000, ALL, 1.0, "fp32c", 16),
    (7 * K + 1, ALL, 1.0, "fp32c", 32), (4 * K, ALL, 1.0, "fp64", 16), (270001, ALL, 1.0, "fp64", 32),
    (16 * K, ALL, 1.0, "fp32c", 32), (24 * K, ALL, 1.0, "fp32c", 64), (16 * K, ALL, 1.0, "fp64", 64),
    # 1024 sources
    (K, 1024, 1.0, "fp32c", 8), (4 * K, 1024, 1.0, "fp32c", 16), (420001, 1024, 1.0, "fp32c", 32),
    (4 * K, 1024, 1.0, "fp64", 16), (4 * K + 1, 1024, 1.0, "fp64", 64), (330001, 4096, 1.0, "fp64", 32),
    # ... at small opening angles
    (K, 1024, 0.3, "fp32c", 8), (200001, 1024, 0.3, "fp32c", 16), (7 * K // 2, 1024, 0.3, "fp32c", 32),
    (4 * K, 1024, 0.3, "fp64", 32), (4 * K, 1024, 0.4, "fp32c", 16), (4 * K, 4096, 0.3, "fp32c", 16),
    (4 * K, 255, 0.3, "fp32c", 16), (330001, 1024, 0.3, "fp32c", 32), (6 * K, 1024, 0.3, "fp32c", 64),
    (6 * K, 64, 0.3, "fp32c", 32), (16 * K, 1024, 0.3, "fp32c", 64), (16 * K, 1024, 0.5, "fp32c", 32),
    # few sources: enough targets for a batch of 64 rays
    (1000, 1, 1.0, "fp32c", 64), (1000, 16, 1.0, "fp32c", 4)])
def test_choice(choose, n, n_src, theta, prec, tile):
    assert choose(n, n_src or n, theta, prec)[0] == tile


@pytest.mark.parametrize("n,n_src,theta,prec,tile", [
    # the smallest opening angle, and the ends of the range of sources
    (4 * K, 1024, 0.0, "fp32c", 16), (4 * K, 1024, 0.0, "fp64", 16), (4 * K, 1024, 0.1, "fp32c", 32),
    (4 * K, 2048, 0.2, "fp32c", 32), (4 * K, 2049, 0.2, "fp32c", 16), (4 * K, 3000, 0.2, "fp64", 16),
    (7 * K, 512, 0.2, "fp32c", 32), (7 * K, 513, 0.2, "fp32c", 64), (8 * K, 512, 0.2, "fp32c", 64),
    (8 * K, 512, 0.0, "fp32c", 64)])
def test_long_lists(choose, n, n_src, theta, prec, tile):
    assert choose(n, n_src, theta, prec)[0] == tile


def test_scenes_of_a_batch(choose):
    assert choose(4 * K, 16384, max_t=16384)[0] == 8
    assert choose(16 * K, 16384, max_t=16384)[0] == 16
    assert choose(64 * K, 16384, max_t=16384)[0] == 64


@pytest.mark.parametrize("n,n_src,grid,prec,tile", [
    # short lists on small grids: the total decides
    (K - 1, 64, 16, "fp32c", 8), (K, 64, 16, "fp32c", 16), (4 * K, 64, 16, "fp32c", 64), (4 * K, 64, 32, "fp32c", 32),
    (4 * K, 64, 32, "fp64", 64), (4 * K, 64, 64, "fp64", 8), (4 * K, 256, 32, "fp32c", 8), (8 * K, 256, 32, "fp32c", 32),
    (8 * K, 1023, 32, "fp64", 64), (8 * K, 1024, 32, "fp64", 8), (64 * K, 256, 32, "fp32c", 64)])
def test_scenes_with_few_sources(choose, n, n_src, grid, prec, tile):
    assert choose(n, n_src, prec=prec, max_t=4096, grid=grid)[0] == tile


def test_size_classes_tell_the_choices_apart(choose):
    """A batch of many small FP32C scenes and one large FP64 call of the same total
    and sources have tiles of their own."""
    base = dict(n=16 * K, n_src=1024, theta=0.5, prec="fp32c")   # on 128^3 cells
    cls = choose(**base)[1]
    assert choose(**{**base, "theta": 0.0})[1] != choose(**{**base, "theta": 0.3})[1]
    for other in (dict(prec="fp64"), dict(theta=0.3), dict(max_t=4096), dict(n=32 * K), dict(n_src=64), dict(grid=32)):
        assert choose(**{**base, **other})[1] != cls, other
