"""The rules by which the fused backward chooses its kernels (csrc/attn_rules.hpp), on the CPU, at calls where both sides were measured."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_09397_amd", "csrc")
SOURCE = """
#include "attn_rules.hpp"
extern "C" int one_launch(int causal, int n, int d, int heads) {
    return attn::own_rows(causal != 0, n, d, 2L * heads * ((n + 63) / 64), false);
}
extern "C" int eight(int causal, int mask_form, int n, int heads) { return attn::eight_waves_bwd(causal != 0, mask_form != 0, n, heads); }
"""
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    folder = tmp_path_factory.mktemp("rules")
    (folder / "rules.cpp").write_text(SOURCE)
    out = str(folder / "rules.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(folder / "rules.cpp"), "-o", out])
    return ctypes.CDLL(out)


@pytest.mark.parametrize("causal,d,heads,n,one", [
    # full attention, more than one block per CU: 10 to 19 % slower in one launch
    (0, 64, 38, 320, 0), (0, 64, 31, 372, 0), (0, 64, 52, 417, 0), (0, 64, 45, 448, 0), (0, 128, 37, 256, 0),
    (0, 64, 17, 448, 1), (0, 64, 31, 200, 1), (0, 64, 62, 200, 1), (0, 64, 80, 200, 0), (0, 64, 47, 256, 0), (0, 128, 31, 256, 1), (0, 256, 30, 64, 1),
    (1, 64, 8, 333, 1), (1, 64, 50, 320, 1), (1, 64, 95, 200, 1), (1, 64, 110, 320, 0), (1, 64, 8, 449, 0), (1, 128, 8, 257, 0),
])
def test_short_calls_in_one_launch(lib, causal, d, heads, n, one):
    assert lib.one_launch(causal, n, d, heads) == one


@pytest.mark.parametrize("causal,mask_form,heads,n,eight_waves", [
    # dQ of the weight gradient, causal, more blocks than CUs: short calls were 5 to 9 % slower with eight waves
    (1, 0, 60, 300, 0), (1, 0, 61, 336, 0), (1, 0, 41, 500, 0), (1, 0, 34, 700, 0), (1, 0, 23, 1024, 0),
    (1, 0, 50, 300, 1), (1, 0, 26, 700, 1), (1, 0, 20, 1024, 1), (1, 0, 18, 1280, 1), (1, 0, 20, 1500, 1), (1, 0, 4, 8192, 1), (1, 0, 22, 1900, 0),
    (1, 1, 16, 700, 1), (1, 1, 16, 1024, 0), (0, 1, 11, 700, 1), (0, 1, 10, 1024, 0), (0, 0, 16, 1024, 1), (0, 0, 12, 1500, 0), (0, 0, 8, 256, 0),
])
def test_eight_waves_for_a_block(lib, causal, mask_form, heads, n, eight_waves):
    assert lib.eight(causal, mask_form, n, heads) == eight_waves
