"""The decode launch's two shapes: one block per wavefront up to 1536 blocks per CU, up to three beyond (csrc/decode_plan.h)."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2604_02715_amd import inputs
from test_gpu_materialize import run_against_model

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")


@pytest.mark.gpu
@pytest.mark.parametrize("n", [7, 8])
@pytest.mark.parametrize("per_wave", ["1", "3"])
def test_either_shape(n, per_wave, monkeypatch):
    # about 8700 blocks an expert (1.411 bytes an element in blocks of 4096), sizes that leave a short last block; three blocks for a
    # wavefront of eight are filled from 18400 blocks on 256 CUs on
    monkeypatch.setenv("FLUXMOE_DECODE_BLOCKS_PER_WAVE", per_wave)
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=8, hidden=4104, ffn=2056, n_slots=8)
    run_against_model(cfg, [(0, [3, 0, 6, 1, 5, 2, 4, 7][:n], [7, 2, 0, 5, 1, 6, 3, 4][:n])])


def test_blocks_of_a_workgroup(tmp_path):
    (tmp_path / "shim.cpp").write_text("""
#include "decode_plan.h"
extern "C" uint64_t per_wg(uint64_t total, uint64_t cus, uint64_t waves, uint64_t asked) { return fluxmoe::decode_per_workgroup(total, cus, waves, asked); }
""")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(tmp_path / "shim.cpp"), "-o", str(tmp_path / "shim.so")], check=True)
    fn = C.CDLL(str(tmp_path / "shim.so")).per_wg
    fn.argtypes, fn.restype = [C.c_uint64] * 4, C.c_uint64
    assert [fn(n, 256, 8, 0) for n in (1, 1100, 70000, 393216, 393217, 1 << 21)] == [8, 8, 8, 8, 24, 24]
    assert [fn(n, 256, 8, 3) for n in (1, 1100, 9 * 768, 18432, 70000)] == [8, 8, 9, 24, 24]      # no CU goes without a workgroup
    assert fn(70000, 256, 4, 1) == 4 and fn(70000, 256, 16, 2) == 32 and fn(70000, 32, 8, 0) == 24
