"""Rows of W per tile of the down projection of two to four token rows (csrc/gemm_plan.h, compiled for the CPU)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_17307_amd", "csrc")
WRAP = """
#include "gemm_plan.h"
extern "C" int rows(int d_model, int mp, int n_cu) { return rs::down_tile_rows(d_model, mp, n_cu); }
"""
# every width the rule is asked for, on 256 CUs: the faster tile of both as measured at 2, 3 and 4 rows
FASTER = {128: 2, 256: 2, 384: 2, 512: 2, 640: 3, 768: 3, 896: 2, 1024: 2, 1152: 3, 1280: 3, 1408: 3, 1536: 3, 1664: 3, 1792: 3, 1920: 3, 2048: 3}


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("down_tiles")
    src, so = d / "wrap.cpp", d / "libdown_tiles.so"
    src.write_text(WRAP)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("mp", [2, 4])
def test_three_rows_a_tile_only_where_the_busiest_cu_pulls_less(lib, mp):
    assert {d: lib.rows(d, mp, 256) for d in FASTER} == FASTER


@pytest.mark.gpu
@pytest.mark.parametrize("d", [640, 896, 1024, 2048])
def test_widths_with_remainders_match_the_oracle(d):
    """Both tiles, widths that are 1 and 2 above a multiple of three, two to four rows.  An O projection of zeros keeps attention out of the result, and
    with it the rounding of K and V, which differs now and then between two right answers."""
    import torch
    import paper_2507_17307_amd as P
    import workloads as W
    from oracle import decoder, router
    from parity import check_invocation
    from workloads.shapes import ModelShape
    shape = ModelShape("narrow", 2, d, 4, 2, 32, 640, 1000, tied_lm_head=False)
    w = W.make_weights(shape, 83, 1)
    for layer in w.layers:
        layer.w_o.zero_()
    gpu, ref = P.Model(w.to("cuda"), max_ctx=16, max_rows=4), decoder.OracleModel(w, 16)
    toks = W.rng.randint(83, 1, 0, 9, 1000).tolist()
    pos = 0
    for n in (2, 3, 4):
        got, lg = gpu.forward_span(toks[pos:pos + n], pos, 0.6, P.RS_SLM, 2.0, want_logits=True)
        torch.cuda.synchronize()
        want = ref.forward(toks[pos:pos + n], pos, logit_scale=2.0)["logits"]
        check_invocation(got[0], lg[0], want, 0.6, router.SLM, where=f"width {d}, {n} rows")
        # fp32 against 64 bits: sums of up to 2048 products, each rounding 2^-24 of a partial sum of random signs (about 1e-6 of the result), a few in a chain
        assert float((lg[0].cpu().double() - want).norm()) <= 2e-5 * float(want.norm())
        pos += n
