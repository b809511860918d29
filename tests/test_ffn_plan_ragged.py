"""Launch plans where H or F is not a multiple of 64 (csrc/ffn_plan.h with FfnShape::ragged), compiled on their own: the
256 x 256 tiles stand in for weight strips."""
import ctypes as C
import os
import random
import subprocess
from types import SimpleNamespace

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")
FIELDS = ("tiled", "halves", "m_tile", "ksplit", "ksplit1", "split_tiles", "tiles_cap", "bytes", "off_h", "off_y")
SHIM = """
#include "ffn_plan.h"
using namespace fluxmoe;
extern "C" void plan(uint64_t E, uint64_t H, uint64_t F, int waves, int ragged, uint32_t T, uint32_t K, uint64_t limit, uint32_t mapped, int split, uint64_t* o) {
    const FfnShape c{E, H, F, 256, waves, ragged != 0};
    const FfnPlan p = split ? plan_ffn(c, T, K, limit, mapped) : plan_ffn_rules(c, T, K, mapped, false, ~0ull);
    %s
}
""" % " ".join("o[%d] = p.%s;" % (i, f) for i, f in enumerate(FIELDS))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("ffn_plan_ragged")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    so = C.CDLL(str(d / "shim.so"))
    u32, u64 = C.c_uint32, C.c_uint64
    so.plan.argtypes = [u64, u64, u64, C.c_int, C.c_int, u32, u32, u64, u32, C.c_int, C.POINTER(u64)]

    def call(T, K, E, H, F, mapped=0, limit=2 ** 64 - 1, waves=2, ragged=True, split=True):
        o = (u64 * len(FIELDS))()
        so.plan(E, H, F, waves, ragged, T, K, limit, mapped, split, o)
        return SimpleNamespace(**dict(zip(FIELDS, o)))
    return call


@pytest.fixture(autouse=True)
def no_overrides(monkeypatch):
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)


def test_random_calls_at_any_buffer_size(plan):
    rng = random.Random(9)
    tiles = kept = 0
    for _ in range(3000):
        E = rng.choice([1, 2, 8, 20, 64, 160, 512])
        H, F = 8 * rng.randrange(1, 640), 8 * rng.randrange(1, 640)
        if rng.random() < 0.3:
            H = 64 * rng.randrange(1, 80)
        K = rng.randrange(1, min(E, 12) + 1)
        c = dict(T=max(1, min(65535, int(2 ** rng.uniform(4, 16)))), K=K, E=E, H=H, F=F, mapped=rng.choice([0, 1, E]), waves=rng.choice([2, 2, 2, 1, 8]))
        best, strips, least = plan(**c), plan(**c, ragged=False), plan(**c, split=False)
        assert least.__dict__ == plan(**c, split=False, ragged=False).__dict__           # what is always enough stays what it was
        if H % 64 == 0 and F % 64 == 0 or c["waves"] != 2:
            assert best.__dict__ == strips.__dict__
        for limit in (2 ** 64 - 1, least.bytes, (least.bytes + best.bytes) // 2, best.bytes):
            p = plan(**c, limit=limit)
            if limit >= least.bytes:
                assert p.bytes <= limit
            if not p.tiled or (H % 64 == 0 and F % 64 == 0):
                continue
            pairs = c["T"] * K
            assert p.m_tile == 256 and not p.halves and p.tiles_cap <= 65535
            assert 1 <= p.ksplit <= max(1, F // 64) and 1 <= p.ksplit1 <= max(1, H // 64)
            assert p.off_y >= p.off_h + pairs * F * 2
            assert p.bytes >= p.off_y + p.ksplit * pairs * H * 4
            assert p.bytes >= p.off_y + (p.ksplit1 * pairs * 2 * F * 4 if p.ksplit1 > 1 else 0)
            q = plan(**c, ragged=False, limit=limit)     # sums no longer than the strips'
            chains = q.ksplit1 * (2 if q.halves else 1)
            assert p.ksplit1 >= chains and (chains == 1 or (p.split_tiles == 2 ** 32 - 1 and H >= 256 * chains))
            assert p.ksplit >= q.ksplit
            tiles += 1
            kept += chains > 1
    assert tiles > 500 and kept > 50


def test_the_line_is_that_of_whole_steps(plan):
    of = lambda T, H, F: (lambda p: (bool(p.tiled), p.m_tile))(plan(T, 2, 8, H, F))
    for T in (256, 440, 480, 520, 560, 4096):
        assert of(T, 4104, 14328) == of(T, 4096, 14336)
    assert of(480, 4104, 14328) == (False, 128) and of(560, 4104, 14328) == (True, 256)


@pytest.mark.parametrize("call", [
    dict(T=2000, K=1, E=1, H=5000, F=1496), dict(T=560, K=2, E=8, H=4400, F=3504), dict(T=881, K=8, E=8, H=928, F=392),
])
def test_tiles_give_way_to_the_strips_with_their_splits_and_halves(plan, call):
    """In the bytes the strips' plan takes, and in a buffer of 32 MiB, a call gets no less than that plan."""
    call = dict(call, mapped=call["E"])
    best, strips = plan(**call), plan(**call, ragged=False)
    assert best.tiled and best.bytes > strips.bytes and (strips.halves or strips.ksplit1 > 1)
    assert plan(**call, limit=strips.bytes).__dict__ == strips.__dict__
    assert plan(**call, limit=32 << 20).__dict__ == plan(**call, limit=32 << 20, ragged=False).__dict__


def test_random_calls_fall_back_on_the_strips_plan(plan):
    rng = random.Random(10)
    strips_taken = 0
    for _ in range(3000):
        E, H, F = rng.choice([1, 2, 8, 20, 64, 160]), 8 * rng.randrange(1, 640), 8 * rng.randrange(1, 640)
        c = dict(T=int(2 ** rng.uniform(5, 15)), K=rng.randrange(1, min(E, 12) + 1), E=E, H=H, F=F, mapped=rng.choice([0, E]))
        strips = plan(**c, ragged=False)
        for limit in (strips.bytes, strips.bytes - 1, strips.bytes + rng.randrange(1 << 24), 32 << 20):
            p, q = plan(**c, limit=limit), plan(**c, limit=limit, ragged=False)
            assert p.tiled or p.__dict__ == q.__dict__
            strips_taken += not p.tiled and bool(plan(**c).tiled)
    assert strips_taken > 100


@pytest.mark.parametrize("call", [dict(T=4390, K=3, E=8, H=1856, F=2632), dict(T=1024, K=2, E=8, H=4104, F=14344), dict(T=333, K=4, E=64, H=2880, F=360),
                                  dict(T=560, K=2, E=8, H=4400, F=3504)])
def test_the_size_query_asks_for_little_more_than_strips_take(plan, call):
    """... and a call in a buffer of that size is accepted; the shared expert's query covers its own plan."""
    from paper_2604_02715_amd import binding as B
    best, strips, least = plan(**call), plan(**call, ragged=False), plan(**call, split=False)
    ctx = B.fluxmoe_create(1, call["E"], call["H"], call["F"], call["E"])
    try:
        asked = B.fluxmoe_ffn_workspace_bytes(ctx, call["T"], call["K"])
        needed = max(strips.bytes, least.bytes)
        assert asked == (max(best.bytes, needed) if best.bytes <= needed + (64 << 20) else needed)
        assert plan(**call, mapped=call["E"], limit=asked).bytes <= asked
        alone = dict(T=call["T"], K=1, E=1, H=call["H"], F=call["F"])
        assert B.fluxmoe_ffn_workspace_bytes(ctx, call["T"], call["K"], True) >= max(asked, plan(**alone, ragged=False).bytes, plan(**alone, split=False).bytes)
    finally:
        B.fluxmoe_destroy(ctx)


@pytest.mark.parametrize("hidden", [64, 72])
def test_rows_of_h_too_long_for_a_tile_of_256_stay_with_the_strips(plan, hidden):
    """256 rows of F BF16 values in 32-bit byte offsets: F below 2^23."""
    assert plan(3000, 1, 1, hidden, 2 ** 23 - 64).m_tile == 256
    p = plan(3000, 1, 1, hidden, 2 ** 23)
    assert not p.tiled and p.m_tile == 128


def test_what_the_plan_report_says(plan):
    """fluxmoe_ffn_plan: the plan of a call with every expert resident and scratch of the size that the query asks for; where H
    or F is no multiple of 64 the strips' plan, which such a call takes or replaces by tiles with no fewer splits."""
    from paper_2604_02715_amd import binding as B
    rng = random.Random(12)
    tiles = strips = 0
    calls = [dict(T=1439, K=8, E=8, H=360, F=360), dict(T=4096, K=2, E=8, H=4096, F=14336), dict(T=1024, K=2, E=8, H=4104, F=14344)]
    for _ in range(300):
        step = rng.choice([8, 64])
        calls.append(dict(T=int(2 ** rng.uniform(4, 13)), K=rng.randrange(1, 9), E=rng.choice([8, 20, 64]), H=step * rng.randrange(1, 2400 // step), F=step * rng.randrange(1, 2400 // step)))
    for c in calls:
        ctx = B.fluxmoe_create(1, c["E"], c["H"], c["F"], c["E"])
        try:
            said, limit = B.fluxmoe_ffn_plan(ctx, c["T"], c["K"]), B.fluxmoe_ffn_workspace_bytes(ctx, c["T"], c["K"])
        finally:
            B.fluxmoe_destroy(ctx)
        p, q = plan(**c, mapped=c["E"], limit=limit), plan(**c, mapped=c["E"], limit=limit, ragged=False)
        assert said == (q.m_tile, q.ksplit)
        if p.__dict__ != q.__dict__:
            assert (c["H"] % 64 or c["F"] % 64) and p.m_tile == 256 and p.ksplit >= q.ksplit
            tiles += 1
        strips += not p.tiled
    assert tiles > 20 and strips > 30


def test_short_k_stays_with_the_strips(plan):
    """Tiles whose K splits stand for the strips' halves: from H 384 a split on, 512 where the sums pass 256 MB."""
    of = lambda T, H, F, K=1, E=8: bool(plan(T, K, E, H, F).tiled)
    assert not of(1460, 528, 2632) and of(2471, 816, 1016) and of(881, 928, 392, K=8)
    assert not of(9395, 608, 896, K=8) and not of(9952, 728, 272, K=8, E=160)
    assert of(10702, 1224, 896, K=2, E=160) and of(6256, 2496, 1400, K=10, E=160)
