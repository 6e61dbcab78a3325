"""The work split of the walked attention (csrc/attn_plan.h), compiled for the CPU."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_17307_amd", "csrc")
WRAP = """
#include "attn_plan.h"
extern "C" int next_pass(int t0, int t_end) { return rs::walk_next_pass(t0, t_end); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("attn_plan")
    src, so = d / "wrap.cpp", d / "libattn_plan.so"
    src.write_text(WRAP)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("t_begin,t_end", [(0, 1), (0, 63), (0, 64), (0, 65), (64, 130), (128, 4562), (4544, 4562), (0, 9157)])
def test_requests_of_a_slice_stay_on_its_pass_grid(lib, t_begin, t_end):
    """Every request starts a whole pass of the slice (16-byte V pieces are aligned there), none lies past the slice, and a
    slice requests each of its passes: once, and the last one once more."""
    starts, t0 = [t_begin], t_begin
    while t0 < t_end:
        starts.append(lib.next_pass(t0, t_end))
        t0 += 64
    passes = list(range(t_begin, t_end, 64))
    assert starts == passes + passes[-1:]
