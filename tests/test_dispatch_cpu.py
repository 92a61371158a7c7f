"""Choices of the launchers that sizes decide (host-only).  No GPU."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    return ctypes.CDLL(os.path.join(ROOT, "paper_2007_01088_amd", "libcc3.so"))


# Time per output of the split-BF16 tiles of edge 64 to 128 relative to 128, measured: a smaller
# edge has to save as much padding.
TIME = {4: 1.4, 5: 1.4, 6: 1.4, 7: 1.1, 8: 1.0}


@pytest.mark.parametrize("nv", [93, 120, 150, 187, 210, 250, 385, 400, 450, 480, 561, 785, 800,
                                897, 930, 960])
def test_small_edges_save_what_they_cost(lib, nv):
    f = lib._ZN3cc313lp_tile_wavesEll
    f.argtypes = [ctypes.c_long] * 2
    nw = f(nv, nv)
    assert 4 <= nw <= 8
    work = lambda n: (-(-nv // (16 * n)) * 16 * n) ** 2 * TIME[n]
    assert work(nw) <= work(8), f"edge {16 * nw} costs more than 128 at nv = {nv}"


@pytest.mark.parametrize("nv,ntri", [(250, 4), (512, 2), (640, 2), (896, 2), (1024, 2), (250, 8),
                                     (120, 32), (20, 16)])
def test_zo_partials_fill_the_chip(lib, nv, ntri):
    chunks = lib._ZN3cc311zo_nbchunksEii(nv, ntri)
    units = nv * (-(-nv // 8))  # of 8 k
    assert 1 <= chunks <= units
    waves = chunks * 3 * -(-nv // 64) * ntri
    assert waves >= 2048 or (chunks + 1) * 64 > units, "two wavefronts per SIMD, or 64 units each"
