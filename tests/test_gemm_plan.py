"""The launch arithmetic of the matrix-core products (csrc/gemm_plan.h), compiled for the CPU."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_17307_amd", "csrc")
WRAP = """
#include "gemm_plan.h"
extern "C" int few(int one_block, int n_tiles, int n_win, int n_cu) { return rs::split_few(one_block, n_tiles, n_win, n_cu); }
extern "C" int many(int n_tiles, int n_win, int n_cu) { return rs::split_many(false, n_tiles, n_win, n_cu).ks; }
extern "C" int ring_layer(int n_cu, int rows, int gateup, int n_out, int K) { return rs::ring_layer(n_cu, rows, gateup, n_out, K); }
extern "C" int tiles(int lm_head, int rows, int n_tiles, int n_win, int ks, int n_cu) { return rs::plan_ring(lm_head, rows, n_tiles, n_win, ks, n_cu); }
extern "C" int ring_lm_head(int n_cu, int n_seqs, int vocab) { return rs::ring_lm_head(n_cu, n_seqs, vocab); }
extern "C" int eight(int lm_head, int rows, int ct) { return rs::ring_eight_waves(lm_head, rows, ct); }
"""
CU = 256
# outputs and width of the products whose K is split
SHAPES = {"s15": (1536, 12, 2, 8960), "m7": (3584, 28, 4, 18944), "m14": (5120, 40, 8, 13824), "m32": (5120, 40, 8, 27648)}


def products(shape):
    d, nq, nkv, ffn = SHAPES[shape]
    return {"qkv": ((nq + 2 * nkv) * 128, d), "o": (d, nq * 128), "down": (d, ffn)}


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("gemm_plan")
    src, so = d / "wrap.cpp", d / "libgemm_plan.so"
    src.write_text(WRAP)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


# workgroup-level splits of K on 256 CUs: up to 16 rows; more rows on k_gemm_rows; more rows on k_gemm_ring (0: does not take it)
SPLITS = {
    ("s15", "qkv"): (4, 4, 0), ("s15", "o"): (4, 4, 0), ("s15", "down"): (8, 8, 8),
    ("m7", "qkv"): (4, 8, 7), ("m7", "o"): (4, 8, 8), ("m7", "down"): (8, 8, 8),
    ("m14", "qkv"): (2, 4, 4), ("m14", "o"): (4, 8, 8), ("m14", "down"): (8, 8, 8),
    ("m32", "qkv"): (2, 4, 4), ("m32", "o"): (4, 8, 8), ("m32", "down"): (8, 8, 8),
}


@pytest.mark.parametrize("shape,name", SPLITS)
def test_the_order_of_sums_of_a_product(lib, shape, name):
    """K and V are rounded to bf16, so the split of a sum can be seen in later logits: what a split is follows from the matrix and the number
    of CUs alone, and which of the two kernels takes up to 16 rows does not matter to it."""
    n, k = products(shape)[name]
    tiles, wins = n // 16, k // 64
    many = [lib.many(tiles, wins, CU) if lib.ring_layer(CU, rows, 0, n, k) else 0 for rows in (17, 64, 65, 128)]
    assert len(set(many)) == 1
    assert (lib.few(1, tiles, wins, CU), lib.few(0, tiles, wins, CU), many[0]) == SPLITS[shape, name]


@pytest.mark.parametrize("rows", [65, 96, 128])
@pytest.mark.parametrize("vocab", [50257, 53248])
def test_lm_head_of_many_sequences_in_one_round(lib, rows, vocab):
    """A vocabulary that 13 tiles a workgroup hold in one round of the machine does not take two."""
    assert lib.tiles(1, rows, (vocab + 15) // 16, 24, 1, CU) == 13


@pytest.mark.parametrize("rows", [18, 40, 65, 128])
def test_the_lm_head_tests_of_thirteen_tiles_take_thirteen(lib, rows):
    """The shape of test_gpu_operand_order.py: 53233 entries, two windows of K."""
    assert lib.tiles(1, rows, (53233 + 15) // 16, 2, 1, CU) == 13


@pytest.mark.parametrize("rows", [81, 97, 128])
def test_the_widest_groups_of_many_rows_are_tested(lib, rows):
    """The shape of test_gpu_gemm_ring.py whose gate/up takes 14 tiles on four waves of two row blocks: X two windows in LDS, W three."""
    assert lib.tiles(0, rows, 27648 // 8, 1536 // 64, 1, CU) == 14 and not lib.eight(0, rows, 14)
    assert lib.ring_layer(CU, rows, 1, 27648, 1536) and lib.ring_layer(CU, rows, 0, 1536, 27648)      # (gate/up and down go together)


@pytest.mark.parametrize("rows", [65, 128])
def test_narrow_groups_of_many_rows_fill_the_machine(lib, rows):
    """The 1.5B shape's down projection above 64 rows: 96 tiles, K split 8 ways, take every CU, and two waves a SIMD."""
    ct = lib.tiles(0, rows, 96, 140, 8, CU)
    assert -(-96 // ct) * 8 == CU and lib.eight(0, rows, ct)


@pytest.mark.parametrize("shape,name,gateup,takes", [
    # rows at which the matrix takes k_gemm_ring, of 4, 5, 8 and 16 (the measurements beside ring_layer)
    ("s15", "gu", 1, ()), ("s15", "down", 0, ()), ("m7", "qkv", 0, ()), ("m7", "o", 0, ()), ("m7", "gu", 1, (4, 5, 8, 16)),
    ("m7", "down", 0, (5, 8, 16)), ("m14", "qkv", 0, ()), ("m14", "o", 0, ()), ("m14", "gu", 1, (4, 5, 8, 16)), ("m14", "down", 0, (4, 5, 8, 16)),
    ("m32", "qkv", 0, ()), ("m32", "gu", 1, (4, 5, 8, 16)), ("m32", "down", 0, (4, 5, 8, 16))])
def test_which_products_of_few_rows_take_the_ring(lib, shape, name, gateup, takes):
    """Not those that k_gemm_rows spreads evenly over the CUs."""
    d, _, _, ffn = SHAPES[shape]
    n, k = (ffn, d) if gateup else products(shape)[name]
    assert tuple(r for r in (4, 5, 8, 16) if lib.ring_layer(CU, r, gateup, n, k)) == takes


def test_the_layer_that_changes_kernels_between_4_and_5_rows(lib):
    """The shape of test_gpu_gemm_ring.py that compares the two kernels' sums, and its LM head on either side of the rule."""
    assert not lib.ring_layer(CU, 4, 0, 3584, 16896) and lib.ring_layer(CU, 5, 0, 3584, 16896)
    assert not lib.ring_lm_head(CU, 3, 20464) and lib.ring_lm_head(CU, 3, 20480)
