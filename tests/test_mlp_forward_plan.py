"""The forward plan of the fp32 row kernel, compiled for the CPU: its loads stay inside the weight copy, every weight is multiplied once,
and the activations that a layer leaves reach as far as the next layer reads."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SIDES = list(range(1, 70)) + [127, 128, 129, 191, 193, 255, 256, 257, 320, 321, 511, 512]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("plan") / "mlp_forward_plan.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "mlp_forward_plan.cpp"), "-o", out],
                   check=True)
    lib = ctypes.CDLL(out)
    lib.f32_forward_reach.restype = ctypes.c_long
    return lib


@pytest.mark.parametrize("head", [False, True])
def test_every_weight_is_loaded_once_from_inside_the_copy(plan, head):
    kp, ldn = ctypes.c_int(), ctypes.c_int()
    for fin in SIDES + [1000, 1024]:
        for fout in [n for n in SIDES if n <= (64 if head else 512)]:
            reach = plan.f32_forward_reach(fin, fout, head, ctypes.byref(kp), ctypes.byref(ldn))
            assert 0 < reach <= kp.value * ldn.value, (fin, fout)
            assert fin <= kp.value <= (fin + 63) // 64 * 64, (fin, fout)   # rows of whole 64 columns hold what is read
            assert ldn.value == (fout + 63) // 64 * 64, (fin, fout)
