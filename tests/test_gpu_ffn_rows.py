"""GPU parity of the walking 256 x 256 tiles that are taken row by row (experts of about one row tile, few column tiles), against the FP64
oracle: more tiles than workgroups, so that workgroups walk on, column tiles that do not divide an XCD's 32, a few tiles only, weights that
pass the caches by.  The plan's rules say that both products take them so."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2604_02715_amd import inputs
from test_ffn_plan import rules  # noqa: F401 (fixture)
from test_gpu_ffn import run_ffn_case

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")
SHIM = """
#include "ffn_plan.h"
extern "C" int rows(uint64_t n_ct, uint64_t avg, uint32_t group) { return fluxmoe::tiles_by_rows(n_ct, avg, group); }
extern "C" int streams(uint64_t e, uint64_t h, uint64_t f, uint64_t pairs) { return fluxmoe::weights_stream(e, h, f, pairs, 256); }
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_order")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    so = C.CDLL(str(d / "shim.so"))
    so.rows.argtypes, so.streams.argtypes = [C.c_uint64] * 2 + [C.c_uint32], [C.c_uint64] * 4
    return so


CASES = [
    # weights pass the caches by, experts, tokens, top_k, hidden, ffn, routing
    (False, dict(n_experts=64, n_slots=64, tokens=8000, top_k=2, hidden=512, ffn=576, routing="uniform")),      # 5 and 2 column tiles, 250 rows each
    (False, dict(n_experts=60, n_slots=60, tokens=6000, top_k=3, hidden=320, ffn=704, routing="zipf")),         # row tiles of 1 to 256 rows, up to dozens for an expert
    (False, dict(n_experts=3, n_slots=3, tokens=520, top_k=1, hidden=128, ffn=64, routing="uniform")),          # one column tile each, fewer tiles than XCDs
    (True, dict(n_experts=64, n_slots=64, tokens=6100, top_k=2, hidden=704, ffn=576, routing="uniform")),       # 156 MB of weights; 5 and 3 column tiles
]


@pytest.mark.parametrize("streams,kw", CASES)
def test_the_rules_take_them_row_by_row(streams, kw, order, rules):  # noqa: F811
    pairs, E, H, F = kw["tokens"] * kw["top_k"], kw["n_experts"], kw["hidden"], kw["ffn"]
    p = rules.plan(T=kw["tokens"], K=kw["top_k"], E=E, H=H, F=F, mapped=E)
    avg = pairs // min(E, pairs)
    assert p.tiled and p.m_tile == 256 and p.ksplit1 == 1
    assert order.rows(-(-F // 128), avg, 0) and order.rows(-(-H // 256), avg, 0) and bool(order.streams(E, H, F, pairs)) == streams
    if streams or E == 64:
        assert p.ksplit == 1                                             # the second product walks too


@pytest.mark.gpu
@pytest.mark.parametrize("streams,kw", CASES)
def test_tiles_row_by_row(streams, kw):
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw), seed=31)


def test_both_sides_of_the_lines(order):
    assert order.rows(24, 384, 0) and not order.rows(25, 384, 0) and not order.rows(24, 385, 0)
    assert not order.rows(24, 384, 2)                                        # a group asked for by FLUXMOE_FFN_TILED_GROUP
