"""The shared expert's launch plan (plan_shared and ring_product in csrc/ffn_plan.h), compiled on its own."""
import ctypes as C
import os
import random
import subprocess
from types import SimpleNamespace

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")
FIELDS = ("tiled", "m_tile", "ring1", "ring2", "ksplit", "ksplit1", "bytes", "off_h", "off_y")
SHIM = """
#include "ffn_plan.h"
using namespace fluxmoe;
static void put(const FfnPlan& p, uint64_t* o) { %s }
extern "C" void shared(uint64_t H, uint64_t F, int n_cus, int waves, uint32_t T, uint64_t limit, uint64_t* o) { put(plan_shared(FfnShape{1, H, F, n_cus, waves, true}, T, limit), o); }
extern "C" void base(uint64_t H, uint64_t F, int n_cus, int waves, uint32_t T, uint64_t limit, uint64_t* o) { put(plan_ffn(FfnShape{1, H, F, n_cus, waves, true, false}, T, 1, limit), o); }
extern "C" uint64_t asked(uint64_t H, uint64_t F, uint32_t T) { return shared_bytes(FfnShape{1, H, F, 256, 2, true}, T); }
extern "C" void least(uint64_t H, uint64_t F, int n_cus, int waves, uint32_t T, uint64_t, uint64_t* o) { put(plan_ffn_rules(FfnShape{1, H, F, n_cus, waves, true}, T, 1, 0, false, ~0ull), o); }
""" % " ".join("o[%d] = p.%s;" % (i, f) for i, f in enumerate(FIELDS))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("ffn_plan_shared")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    so = C.CDLL(str(d / "shim.so"))

    def call(name):
        fn = getattr(so, name)
        fn.argtypes = [C.c_uint64, C.c_uint64, C.c_int, C.c_int, C.c_uint32, C.c_uint64, C.POINTER(C.c_uint64)]

        def f(T, H, F, limit=2 ** 64 - 1, n_cus=256, waves=2):
            o = (C.c_uint64 * len(FIELDS))()
            fn(H, F, n_cus, waves, T, limit, o)
            return SimpleNamespace(**dict(zip(FIELDS, o)))
        return f
    so.asked.argtypes, so.asked.restype = [C.c_uint64] * 2 + [C.c_uint32], C.c_uint64
    return SimpleNamespace(asked=so.asked, **{n: call(n) for n in ("shared", "base", "least")})


@pytest.fixture(autouse=True)
def no_overrides(monkeypatch):
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)


def test_random_shapes_at_any_buffer_size(rules):
    """What launch_ring requires holds, the scratch covers what the kernels write, and a buffer that was enough without the ring
    kernel still is."""
    rng = random.Random(3)
    ring = split = 0
    for _ in range(3000):
        T, H, F = int(2 ** rng.uniform(0, 16)) or 1, 8 * rng.randrange(1, 700), 8 * rng.randrange(1, 900)
        T = min(T, 65535)
        waves, n_cus = rng.choice([2, 2, 2, 1, 8]), rng.choice([256, 256, 304, 32])
        best, least = rules.shared(T, H, F, n_cus=n_cus, waves=waves), rules.least(T, H, F, n_cus=n_cus, waves=waves)
        for limit in (2 ** 64 - 1, least.bytes, (least.bytes + best.bytes) // 2, best.bytes, least.bytes + rng.randrange(1 << 20)):
            p, b = rules.shared(T, H, F, limit, n_cus, waves), rules.base(T, H, F, limit, n_cus, waves)
            if limit >= least.bytes:
                assert p.bytes <= limit and b.bytes <= limit
            if not p.ring1:
                assert vars(p) == vars(b)
                continue
            assert waves == 2 and p.ring1 in (32, 64, 128) and p.ring2 in (32, 64, 128) and not p.tiled
            assert 1 <= p.ksplit1 <= -(-H // 64) and 1 <= p.ksplit <= -(-F // 64)
            assert p.off_y >= p.off_h + T * F * 2
            assert p.bytes >= p.off_y + (p.ksplit1 * T * 2 * F * 4 if p.ksplit1 > 1 else 0)
            assert p.bytes >= p.off_y + (p.ksplit * T * H * 4 if p.ksplit > 1 else 0)
            ring += 1
            split += p.ksplit1 > 1 or p.ksplit > 1
    assert ring > 2000 and split > 500


def test_where_the_ring_kernel_ends(rules):
    of = lambda T, H=5120, F=1536, **kw: (lambda p: (p.ring1, p.ksplit1, p.ring2, p.ksplit))(rules.shared(T, H, F, **kw))
    assert of(512) == (128, 2, 128, 1)
    assert of(768)[0] == 128 and of(769)[0] == 0                             # second product: 240 workgroups of 128 rows, 280
    assert of(1024, F=384)[0] == 128 and of(1024, F=1024)[0] == 0            # two short rounds, two long ones
    assert of(704, 4504, 2776)[0] == 64 and of(705, 4504, 2776)[0] == 0      # not whole steps: 484 workgroups of 64 rows, 528
    assert of(128, 4096, 14336)[0] == 128 and of(129, 4096, 14336)[0] == 0   # 224; 448 of 128 rows, 672 of 64
    assert of(512, waves=1)[0] == 0


def test_only_the_larger_partial_sums_give_way(rules):
    """17 rows of H 2360 F 1848: eight splits of the second product fill the scratch, five of the first do not."""
    best = rules.shared(17, 2360, 1848)
    assert best.ring1 and best.ksplit1 == 5 and best.ksplit == 8
    p = rules.shared(17, 2360, 1848, best.bytes - 1)
    assert p.ring1 and p.ksplit1 == 5 and p.ksplit == 7 and p.bytes < best.bytes


def test_the_query_asks_for_nothing_that_only_routed_calls_use(rules):
    """H and F of whole steps and neither product split: the scratch is h and one set of sums."""
    rng = random.Random(4)
    seen = 0
    for T, H, F in [(8192, 4096, 4096), (8192, 4096, 14336)] + [(rng.randrange(1, 16000), 64 * rng.randrange(1, 80), 64 * rng.randrange(1, 120)) for _ in range(2000)]:
        p, least = rules.shared(T, H, F), rules.least(T, H, F)
        if not p.ring1 and p.ksplit == p.ksplit1 == 1:
            assert rules.asked(H, F, T) <= max(p.off_y + T * H * 4, least.bytes) + 256
            seen += T > 2000
    assert seen > 200
