"""The choice between the matrix kernels, compiled for the CPU: each shape takes the kernel that is faster there."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("plan") / "gemm_plan.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "gemm_plan.cpp"), "-o", out],
                   check=True)
    return ctypes.CDLL(out)


def _up(n, d=256):
    return (n + d - 1) // d


def _pair_tiles(width, batch):
    """Tiles of a hidden layer's weight gradient (a slice per 1024 rows, at most eight) and input gradient."""
    return _up(width) ** 2 * max(1, min(8, batch // 1024)) + _up(width) * _up(batch)


# widths and batches at which the gradients of three such layers are faster on 256 x 128 tiles, and on 256 x 256
@pytest.mark.parametrize("width,batch,wide", [
    (256, 32768, False), (300, 12288, False), (384, 24576, False), (512, 12288, False), (512, 32768, False), (640, 12288, False),
    (832, 4096, False), (1024, 4096, False), (832, 4608, False),
    (704, 16384, True), (768, 12288, True), (900, 8192, True), (1024, 5120, True), (1024, 8192, True), (1024, 32768, True),
    (1280, 4096, True),
])
def test_gradients_of_hidden_layers_take_the_faster_tiles(plan, width, batch, wide):
    assert plan.wide_pair_pays(_pair_tiles(width, batch), _up(width, 64) * 64) == wide


# (width, inputs, rows under the online weights, rows under the target's)
@pytest.mark.parametrize("width,k,rows,wide", [
    (512, 512, (8192, 0), False), (1024, 1024, (4096, 0), False),                            # a quarter of a round
    (520, 5184, (4096, 2048), False), (640, 3136, (4096, 2048), False), (1032, 3136, (4096, 2048), False),   # halves, long
    (576, 576, (32768, 0), False), (768, 768, (32768, 0), False), (640, 640, (21760, 10880), False),          # two rounds of halves
    (768, 768, (24576, 0), True), (1024, 1024, (24576, 0), True), (512, 512, (49152, 0), True),
    (704, 704, (4096, 2048), True), (768, 768, (6000, 3000), True), (1024, 1024, (12288, 0), True),
    (1024, 3136, (6000, 3000), True), (2048, 3136, (8192, 4096), True),
])
def test_forward_passes_take_the_faster_tiles(plan, width, k, rows, wide):
    assert plan.wide_forward_pays(_up(width), sum(_up(r) for r in rows), k) == wide


def _busiest_xcd(tiles_i, tiles_j, whole):
    """Time of the busiest of eight XCDs of 32 units, in half tiles: a column's tiles go to XCD (column % 8), whole ones first."""
    most = 0
    for xcd in range(8):
        n_whole = tiles_i * len(range(xcd, whole, 8))
        n_half = tiles_i * len(range(xcd, 2 * (tiles_j - whole), 8))
        units = [0] * 32
        for n, cost in ((n_whole, 2), (n_half, 1)):
            for _ in range(n):
                units.sort()
                units[0] += cost
        most = max(most, max(units))
    return most


def test_columns_cut_into_halves_leave_no_xcd_behind(plan):
    for tiles_i in range(1, 9):
        for tiles_j in range(1, 700 // tiles_i):
            rest = tiles_i * tiles_j % 256
            whole = plan.wide_whole_columns(tiles_i, tiles_j)
            assert (whole == tiles_j) == (rest == 0 or rest > 128) and 0 <= whole <= tiles_j
            if whole < tiles_j:
                assert _busiest_xcd(tiles_i, tiles_j, whole) <= _busiest_xcd(tiles_i, tiles_j, (tiles_i * tiles_j - rest) // tiles_i)
    # 640 units at 32768 rows: half a round behind one whole round, on every XCD
    assert _busiest_xcd(3, 128, plan.wide_whole_columns(3, 128)) == 3


# (observation, width, head outputs, most rows) of 256 x 128 tiles
@pytest.mark.parametrize("dim,width,out,rows,slices", [
    (256, 1024, 32, 8192, 8), (256, 1024, 32, 32768, 16), (640, 1024, 18, 9216, 8), (200, 640, 18, 512, 2),      # XCDs share rows
    (300, 900, 18, 32768, 12), (512, 1024, 18, 32768, 12), (200, 640, 18, 14336, 14), (128, 512, 18, 20480, 20),  # blocks count for more
    (4096, 4096, 18, 32768, 8),                                                                                    # more tiles than the chip
])
def test_slices_of_the_first_and_last_layers_gradients(plan, dim, width, out, rows, slices):
    tiles = _up(dim) * _up(width, 128) + _up(width) * _up(out, 128)
    assert plan.ends_slices(tiles, rows, max(1, min(8, rows // 1024))) == slices
