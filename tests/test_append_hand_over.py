"""A bulk append in one launch: no workgroup may read its sequence's length after another one has advanced it, whenever it
starts.  Followed on the host (append_model.cpp) with the launcher's and the kernel's own arithmetic."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MANY = 1 << 30        # scratch for any number of partial sums


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("append") / "append_model.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "append_model.cpp"), "-o", lib], check=True)
    m = ctypes.CDLL(lib)
    m.append_model.argtypes = [ctypes.c_int] * 4 + [ctypes.c_int64] * 2 + [ctypes.c_int]
    m.append_workgroups.argtypes = [ctypes.c_int] * 2 + [ctypes.c_int64] * 2
    return m


@pytest.mark.parametrize("d_h", [64, 128, 256])
@pytest.mark.parametrize("heads,held", [(1, MANY), (8, MANY), (60, MANY), (2, 3), (5, 1)])
def test_a_late_workgroup_sees_the_old_length(model, d_h, heads, held):
    for n_new, step in ((2, 1), (63, 1), (100, 1), (129, 2), (513, 13), (1024, 97), (8191, 1021)):
        for S in (0, 1, 7, 8, 60, 63, 64, 65, 100, 127, 1000, 4095):
            assert model.append_model(S, n_new, step, d_h, heads, held, 0) == 0, (S, n_new)


def test_the_model_notices_workgroups_that_are_not_counted(model):
    """100 rows behind an empty cache: two workgroups of 128 positions, the second without rows; counted only when it has
    some, it finds the new length when it starts late and writes rows 92 .. 99 a second time."""
    assert model.append_workgroups(100, 128, 8, MANY) == 2
    assert model.append_model(0, 100, 100, 128, 8, MANY, 1) == 1
    assert model.append_model(0, 100, 100, 128, 8, MANY, 0) == 0
