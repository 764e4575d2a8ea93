"""Host-side rules of the spread forward pass (csrc/few_plan.hpp, plain C++), compiled here and checked without a GPU."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_15773_amd", "csrc")
SHIM = """
#include "few_plan.hpp"
using namespace tsdp;
extern "C" {
int safe_rows(int own, int B, int R_cap) { return few_safe_rows(own != 0, B, R_cap); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = tmp_path_factory.mktemp("few_plan")
    src, lib = str(out / "shim.cpp"), str(out / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    return C.CDLL(lib)


def test_rows_of_a_callers_buffer_are_not_read_beyond_the_live_ones(plan):
    # a workgroup of row r loads r ahead of the live row count when r < safe_rows; a caller's buffer may end at the live
    # rows, of which there are fewer than environments once some have finished
    for B in (1, 3, 8):
        for R_cap in (1, B, 5 * B):
            for live in range(R_cap + 1):
                early = [r for r in range(R_cap) if r < plan.safe_rows(0, B, R_cap)]
                assert all(r < live for r in early), (B, R_cap, live)
            assert plan.safe_rows(1, B, R_cap) <= R_cap           # the context's own buffers hold R_cap rows
