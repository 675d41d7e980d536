import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def orc():
    from oracle import orc as _orc

    _orc.lib()
    return _orc


def _plan(tmp_path_factory, name):
    out = str(tmp_path_factory.mktemp("plan") / (name + ".so"))
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), name + ".cpp")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", src, "-o", out], check=True)
    return ctypes.CDLL(out)


@pytest.fixture(scope="session")
def mlp_plan(tmp_path_factory):
    """The plans of the whole-network kernels, compiled for the CPU."""
    return _plan(tmp_path_factory, "mlp_plan")


@pytest.fixture(scope="session")
def tower_plan(tmp_path_factory):
    """The plans of the three convolutions in one kernel, compiled for the CPU."""
    return _plan(tmp_path_factory, "tower_plan")
