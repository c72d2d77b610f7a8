"""Division by a launch constant as a multiplication (csrc/params.h), on the host."""
import ctypes
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2312_04985_amd", "csrc")


@pytest.fixture(scope="module")
def divide(tmp_path_factory):
    d = tmp_path_factory.mktemp("divider")
    src, lib = str(d / "divider.cpp"), str(d / "divider.so")
    with open(src, "w") as f:
        f.write('#include "params.h"\nextern "C" int divide(int n, int d) { return sparq::divided(n, sparq::make_divider(d)); }\n')
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", rocm + "/include",
                    src, "-o", lib], check=True)
    m = ctypes.CDLL(lib)
    m.divide.argtypes = [ctypes.c_int, ctypes.c_int]
    return m.divide


def test_divided_is_the_quotient(divide):
    rng = random.Random(1)
    most = 2 ** 31 - 1
    ds = list(range(1, 300)) + [2 ** i + j for i in range(9, 31) for j in (-1, 0, 1)] + [most] + [rng.randint(1, most) for _ in range(200)]
    for d in ds:
        q = most // d
        ns = {0, 1, d - 1, d, most, most - 1, q * d, q * d - 1} | {k * d + j for k in (1, 2, 3, q // 2) for j in (-1, 0, 1)}
        ns |= {rng.randint(0, most) for _ in range(20)}
        for n in ns:
            if 0 <= n <= most:
                assert divide(n, d) == n // d, (n, d)
