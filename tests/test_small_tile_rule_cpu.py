"""The shape of the small tiles (the library's own rule, called without a GPU).
CPU only."""
from __future__ import annotations

import ctypes as C
import os

import pytest

from paper_1102_1343_amd import fire as F

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1102_1343_amd", "libfire_gfx950.so")
F32, F64 = F.FIRE_F32, F.FIRE_F64


@pytest.fixture(scope="module")
def rule():
    if not os.path.exists(LIB):
        pytest.skip("library not built (run __graft_entry__.build())")
    fn = C.CDLL(LIB)["_ZN4fire9step_kindEPK9fire_meshiPiS3_"]

    def call(sizes, dtype, sr=(10, 10)):
        ms = (F.fire_mesh * len(sizes))(*[F.fire_mesh(nx, ny, 6.0, 6.0, *sr, dtype, 0)
                                          for nx, ny in sizes])
        x, y = C.c_int(), C.c_int()
        return (x.value, y.value) if fn(ms, len(sizes), C.byref(x), C.byref(y)) else None
    return call


def _tiles(sizes, x, y):
    return sum(-(-nx // x) * -(-ny // y) for nx, ny in sizes)


def test_many_members_do_not_grow_the_tile_past_a_member(rule):
    """No shape gives 1 000 members fewer than 1 000 work-groups."""
    for dtype in (F32, F64):
        for side in (8, 20, 19):
            x, y = rule([(side, side)] * 1000, dtype)
            up = -(-side // 10) * 10
            assert x <= up and y <= up


@pytest.mark.parametrize("dtype", [F32, F64])
def test_strips_grow_along_their_length(rule, dtype):
    x, y = rule([(160000, 2)], dtype)
    assert y == 10 and x >= 10
    x, y = rule([(2, 160000)], dtype)
    assert x == 10 and y >= 10
    # two long rows need no more work-groups than threads that own a node do
    x, y = rule([(325000, 2)], F32)
    assert y == 10 and x > 60


@pytest.mark.parametrize("side", [40, 128, 300, 400, 500, 600, 632])
@pytest.mark.parametrize("sr", [(10, 10), (4, 4), (8, 5), (1, 1), (5, 7), (16, 12)])
def test_double_precision_tiles_fit_the_waves_of_a_cu(rule, side, sr):
    """20 waves of the FP64 kernel fit a CU: tiles of four waves or fewer, of
    which five fit, or the smallest tile, where that has more."""
    x, y = rule([(side, side)], F64, sr)
    waves = -(-(x + 4) * (y + 4) // 64)
    least = tuple(-(-8 // s) * s for s in sr)
    assert x % sr[0] == 0 and y % sr[1] == 0
    assert waves <= 4 or (x, y) == least


@pytest.mark.parametrize("sr", [(1, 1), (4, 4), (8, 5), (10, 10), (16, 12), (61, 26), (122, 42)])
@pytest.mark.parametrize("sizes", [[(2, 2)], [(128, 128)], [(517, 389)], [(632, 632)],
                                   [(806, 806)], [(20, 900), (900, 20)], [(64, 64)] * 90])
def test_tiles_hold_what_the_kernel_assumes(rule, sizes, sr):
    """Whole atmosphere cells, one or two nodes per thread of at most 1024
    threads, 64 KiB of LDS with 256 fuels, or the tiled kernel."""
    for dtype, most, size in ((F32, 2048, 4), (F64, 1024, 8)):
        if dtype == F64 and sr[1] > 26:
            continue
        got = rule(sizes, dtype, sr)
        if got is None:
            assert (-(-8 // sr[0]) * sr[0] + 4) * (-(-8 // sr[1]) * sr[1] + 4) > most \
                or sum(a * b for a, b in sizes) > 400000
            continue
        x, y = got
        frame = (x + 6) * (y + 6)
        s1 = (x + 4) * (y + 4)
        npt = 1 if s1 <= 1024 else 2
        nt = -(-(-(-s1 // npt)) // 64) * 64
        assert x % sr[0] == 0 and y % sr[1] == 0
        assert s1 <= most and nt <= 1024 and frame <= (npt + 2) * nt
        assert (3 * frame + 256 * 12 + x * y) * size + 16 <= 65536


def test_line_between_the_kernels(rule):
    assert rule([(632, 632)], F64) and rule([(632, 633)], F64) is None
    assert rule([(806, 806)], F32) and rule([(807, 806)], F32) is None
    assert rule([(632, 316)] * 2, F32) and rule([(632, 317)] * 2, F32) is None
