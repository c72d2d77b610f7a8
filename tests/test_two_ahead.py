"""The order of Step 1b's requests (csrc/two_ahead.h), followed on the host."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2312_04985_amd", "csrc")
SOURCE = """
#include "two_ahead.h"
// requests made, or -1: an item used out of order, from the wrong buffer or from one that was requested anew
extern "C" int follow(int items, int several, int* between_at, int* most_in_flight) {
  int next = 0, used = 0, made = 0, holds[2] = {-1, -1};
  bool right = true;
  *between_at = -1; *most_in_flight = 0;
  sparq::two_ahead(items, several != 0,
                   [&](auto b) { right = right && holds[b.value] < 0; holds[b.value] = next++; ++made;
                                 if (next - used > *most_in_flight) *most_in_flight = next - used; },
                   [&](auto b) { right = right && holds[b.value] == used; holds[b.value] = -1; ++used; },
                   [&]() { right = right && *between_at < 0 && used == 0; *between_at = made; },
                   [&]() { next = 0; holds[1] = -1; });
  return right && used == items ? made : -1;
}
"""


@pytest.fixture(scope="module")
def follow(tmp_path_factory):
    d = tmp_path_factory.mktemp("two_ahead")
    src, lib = str(d / "order.cpp"), str(d / "order.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", rocm + "/include",
                    src, "-o", lib], check=True)
    fn = ctypes.CDLL(lib).follow

    def run(items, several):
        at, most = ctypes.c_int(), ctypes.c_int()
        return fn(items, several, ctypes.byref(at), ctypes.byref(most)), at.value, most.value
    return run


@pytest.mark.parametrize("items", range(0, 25))
def test_every_item_is_requested_once_and_used_in_order(follow, items):
    made, at, most = follow(items, int(items > 1))
    assert made == items and at == min(items, 2) and most == min(items, 2)


def test_threads_of_a_wave_that_has_more_items(follow):
    assert follow(0, 1)[:2] == (0, 0)
    assert follow(1, 1)[:2] == (2, 2)          # the one item a second time
