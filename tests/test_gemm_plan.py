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
    (704, 704, (4096, 2048), True), (768, 768, (6000, 3000), True), (1024, 1024, (12288, 0), True),
    (1024, 3136, (6000, 3000), True), (2048, 3136, (8192, 4096), True),
])
def test_forward_passes_take_the_faster_tiles(plan, width, k, rows, wide):
    assert plan.wide_forward_pays(_up(width) * sum(_up(r) for r in rows), k) == wide
