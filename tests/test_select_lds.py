"""The LDS of the digit-bucket plan's second launch (csrc/params.h), on the host."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2312_04985_amd", "csrc")
SOURCE = """
#include "params.h"
using namespace sparq;
extern "C" void layout(int d_h, int span_len, int n_span, int cand_cap, int* out) {
  const BkSelectLds l = bk_select_lds(d_h, span_len, n_span, cand_cap);
  const int at[] = {l.keyval, l.list, l.bitmap, l.ckey, l.cpos, l.hist, l.tab, l.above, l.with, l.before, l.taken, l.offs, l.part,
                    l.red, l.wcnt, l.ctl, l.words};
  for (int i = 0; i < 17; ++i) out[i] = at[i];
}
"""


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    d = tmp_path_factory.mktemp("select_lds")
    src, lib = str(d / "layout.cpp"), str(d / "layout.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", rocm + "/include",
                    src, "-o", lib], check=True)
    fn = ctypes.CDLL(lib).layout
    out = (ctypes.c_int * 17)()

    def at(*shape):
        fn(*shape, out)
        return list(out)
    return at


@pytest.mark.parametrize("d_h", [64, 128, 256])
@pytest.mark.parametrize("cand_cap", [2048, 4096, 8192])
def test_arrays_lie_apart_and_the_histogram_on_16_bytes(layout, d_h, cand_cap):
    """Every span the plan can give (a multiple of 64 positions up to 8192), from 1 to 64 of them."""
    for span_len in range(64, 8192 + 1, 64):
        for n_span in (1, 2, 15, 16, 17, 63, 64):
            at = layout(d_h, span_len, n_span, cand_cap)
            sizes = [span_len, span_len, span_len // 32, cand_cap, cand_cap, 2048, max(33 * n_span, 512), n_span, n_span, 65, n_span,
                     n_span + 1, 8 * (d_h + 2), 32, 16, 16]
            assert at[0] == 0 and all(b >= a + n for a, b, n in zip(at, at[1:], sizes)), (span_len, n_span, at)
            assert at[5] % 4 == 0, (span_len, n_span, at[5])      # the threshold search reads it in 16-byte pieces
