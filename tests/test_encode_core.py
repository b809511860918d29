"""The offline encoder's loops (csrc/encode_core.h), compiled on their own: the vector forms plan and write the same blocks as
the plain ones, whatever the code and the contents."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")
SHIM = """
#include "encode_core.h"
using namespace fluxmoe;
extern "C" int available() { return encode_vector_available(); }
extern "C" void histogram(const uint16_t* w, uint64_t n, uint64_t* h) { count_exponents(w, n, h); }
extern "C" int64_t encode(const uint16_t* w, uint64_t n, const uint8_t* lens, const uint16_t* codes, int vector, uint8_t* dst, uint32_t* first) {
    const Coder c(lens, codes);
    std::vector<uint32_t> f;
    plan_tensor(w, n, c, 4096, f, vector != 0);
    for (size_t i = 0; i < f.size(); ++i) first[i] = f[i];
    const size_t nb = f.size() - 1, half = nb / 2;
    encode_blocks(w, f, half, nb, c, 4096, dst, vector != 0);
    encode_blocks(w, f, 0, half, c, 4096, dst, vector != 0);
    return int64_t(nb);
}
"""


@pytest.fixture(scope="module")
def core(tmp_path_factory):
    d = tmp_path_factory.mktemp("encode_core")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    so = C.CDLL(str(d / "shim.so"))
    so.encode.restype = C.c_int64
    so.encode.argtypes = [C.c_void_p, C.c_uint64, C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_void_p]
    so.histogram.argtypes = [C.c_void_p, C.c_uint64, C.c_void_p]
    return so


def canonical(lens):
    codes, nxt, prev = np.zeros(256, np.uint16), 0, None
    for length, s in sorted((int(l), s) for s, l in enumerate(lens) if l):
        nxt = 0 if prev is None else (nxt + 1) << (length - prev)
        codes[s], prev = nxt, length
    return codes


CODES = {
    "one symbol": {127: 1},
    "eight bits for all": {s: 8 for s in range(256)},
    "up to twelve bits": {**{120 + i: i + 1 for i in range(11)}, 0: 12, 255: 12},
    "skewed": {**{s: 4 for s in range(112, 124)}, **{s: 6 for s in range(124, 136)}, **{s: 12 for s in range(0, 100)}},
}


@pytest.mark.parametrize("name", list(CODES))
@pytest.mark.parametrize("n", [64, 2944, 2944 + 64, 64 * 1001])
def test_vector_and_plain_forms_agree(core, name, n):
    if not core.available():
        pytest.skip("this processor has no AVX-512 VBMI: only the plain form runs here")
    lens = np.zeros(256, np.uint8)
    for s, l in CODES[name].items():
        lens[s] = l
    codes = canonical(lens)
    rng = np.random.default_rng(n)
    used = np.flatnonzero(lens)
    p = 0.5 ** lens[used].astype(float)
    runs = [rng.choice(used, n, p=p / p.sum()), np.full(n, used[-1]), np.full(n, used[np.argmax(lens[used])])]
    for e in runs:                                           # drawn by the code's own probabilities; one symbol only; the longest code only
        w = (rng.integers(0, 2, n) << 15 | e.astype(np.int64) << 7 | rng.integers(0, 128, n)).astype(np.uint16)
        got = []
        for vector in (0, 1):
            dst, first = np.full((n // 64 + 1) * 4096 + 64, 0xAA, np.uint8), np.zeros(n // 64 + 2, np.uint32)
            nb = core.encode(w.ctypes.data, n, lens.ctypes.data, codes.ctypes.data, vector, dst.ctypes.data, first.ctypes.data)
            assert bool((dst[nb * 4096:] == 0xAA).all())     # nothing past the last block
            got.append((nb, dst.tobytes(), first.tobytes()))
        assert got[0] == got[1]


@pytest.mark.parametrize("n", [1, 7, 8, 63, 100000])
def test_histogram(core, n):
    w = np.random.default_rng(n).integers(0, 65536, n).astype(np.uint16)
    h = np.ones(256, np.uint64)
    core.histogram(w.ctypes.data, n, h.ctypes.data)
    assert np.array_equal(h - 1, np.bincount((w >> 7) & 0xFF, minlength=256).astype(np.uint64))
