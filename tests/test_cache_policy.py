"""What passes the caches by (combine_streams, weights_stream in csrc/ffn_plan.h), compiled on its own."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")


SHIM = """
#include "ffn_plan.h"
extern "C" int streams(uint64_t b, uint64_t m, uint64_t e) { return fluxmoe::combine_streams(b, m, e); }
extern "C" int weights(uint64_t e, uint64_t h, uint64_t f, uint64_t pairs, uint64_t m_tile) { return fluxmoe::weights_stream(e, h, f, pairs, m_tile); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("cache_policy")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    so = C.CDLL(str(d / "shim.so"))
    so.streams.argtypes, so.weights.argtypes = [C.c_uint64] * 3, [C.c_uint64] * 5
    return so


def test_the_sums_that_are_there_decide(rules):
    streams = rules.streams
    line = 256 << 20
    assert not streams(line, 8, 8) and streams(line + 8, 8, 8) and streams(line + 8, 0, 8)       # the whole layer; not known
    sums = 4096 * 8 * 5120 * 4                                                                   # 671 MB for all pairs
    assert streams(sums, 160, 160) and streams(sums, 80, 160) and not streams(sums, 40, 160)
    assert not streams(2 ** 63, 1, 2 ** 40)


def test_weights_that_the_cache_may_hold_are_read_from_there(rules):
    assert rules.weights(8, 4096, 14336, 2000, 256) and not rules.weights(8, 4096, 14336, 8192, 256)      # a tile each, several
    assert not rules.weights(32, 1024, 256, 2400, 128) and rules.weights(32, 2048, 512, 6400, 256)        # 50 MB, 201 MB
    assert not rules.weights(160, 5120, 1536, 20000, 256)                                                 # many experts: skew
