"""When the kernel that adds up the experts' rows passes the caches by (combine_streams in csrc/ffn_plan.h), compiled on its own."""
import ctypes as C
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")


def test_the_sums_that_are_there_decide(tmp_path):
    (tmp_path / "shim.cpp").write_text('#include "ffn_plan.h"\nextern "C" int streams(uint64_t b, uint64_t m, uint64_t e) { return fluxmoe::combine_streams(b, m, e); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(tmp_path / "shim.cpp"), "-o", str(tmp_path / "shim.so")], check=True)
    streams = C.CDLL(str(tmp_path / "shim.so")).streams
    streams.argtypes = [C.c_uint64] * 3
    line = 256 << 20
    assert not streams(line, 8, 8) and streams(line + 8, 8, 8) and streams(line + 8, 0, 8)       # the whole layer; not known
    sums = 4096 * 8 * 5120 * 4                                                                   # 671 MB for all pairs
    assert streams(sums, 160, 160) and streams(sums, 80, 160) and not streams(sums, 40, 160)
    assert not streams(2 ** 63, 1, 2 ** 40)
