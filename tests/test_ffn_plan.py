"""The launch plan of the expert FFN (host arithmetic, csrc/ffn_plan.h), compiled on its own: what the kernels and their
launcher require of a plan, scratch that gives way to the caller's buffer, and the rules on both sides of their lines,
also for the residency counts and buffer sizes that only a call knows."""
import ctypes as C
import os
import random
import subprocess
from types import SimpleNamespace

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")
FIELDS = ("tiled", "halves", "g1_xcd", "m_tile", "ksplit", "ksplit1", "split_tiles", "pairs_cap", "tiles_cap", "n_chunks", "bytes",
          "off_count", "off_offset", "off_sorted", "off_pos", "off_tile", "off_ntiles", "off_h", "off_y")
SHIM = """
#include "ffn_plan.h"
using namespace fluxmoe;
static void put(const FfnPlan& p, uint64_t* o) { %s }
extern "C" void plan(uint64_t E, uint64_t H, uint64_t F, int n_cus, int waves, uint32_t T, uint32_t K, uint64_t limit, uint32_t mapped, uint64_t* o) {
    put(plan_ffn(FfnShape{E, H, F, n_cus, waves}, T, K, limit, mapped), o);
}
extern "C" uint32_t least_cost(uint32_t H, uint32_t F, uint32_t n_cus, uint32_t n_tiles, uint32_t rows, uint32_t most) {
    uint32_t best = 1;
    for (uint32_t k = 2; k <= most; ++k) if (tiled_cost(SplitShape{H, F, n_cus}, n_tiles, rows, k) < tiled_cost(SplitShape{H, F, n_cus}, n_tiles, rows, best)) best = k;
    return best;
}
extern "C" void plain(uint64_t E, uint64_t H, uint64_t F, int n_cus, int waves, uint32_t T, uint32_t K, uint32_t mapped, uint64_t* o) {
    put(plan_ffn_rules(FfnShape{E, H, F, n_cus, waves}, T, K, mapped, false, ~0ull), o);
}
""" % " ".join("o[%d] = p.%s;" % (i, f) for i, f in enumerate(FIELDS))
NO_LIMIT = 2 ** 64 - 1


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("ffn_plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    so = C.CDLL(str(d / "shim.so"))
    u32, u64, out = C.c_uint32, C.c_uint64, C.c_uint64 * len(FIELDS)
    so.plan.argtypes = [u64, u64, u64, C.c_int, C.c_int, u32, u32, u64, u32, C.POINTER(u64)]
    so.plain.argtypes = [u64, u64, u64, C.c_int, C.c_int, u32, u32, u32, C.POINTER(u64)]

    def plan(T, K, E, H, F, mapped=0, limit=NO_LIMIT, waves=2, n_cus=256):
        o = out()
        so.plan(E, H, F, n_cus, waves, T, K, limit, mapped, o)
        return SimpleNamespace(**dict(zip(FIELDS, o)))

    def plain(T, K, E, H, F, mapped=0, waves=2, n_cus=256):
        o = out()
        so.plain(E, H, F, n_cus, waves, T, K, mapped, o)
        return SimpleNamespace(**dict(zip(FIELDS, o)))
    return SimpleNamespace(plan=plan, plain=plain, least_cost=so.least_cost)


@pytest.fixture(autouse=True)
def no_overrides(monkeypatch):
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)


def random_call(rng):
    E = rng.choice([1, 1, 2, 8, 20, 64, 160, 512, 4096])
    H, F = (rng.choice([64, 128]) * rng.randrange(1, 65) if rng.random() < 0.6 else 8 * rng.randrange(1, 640) for _ in range(2))
    K = rng.randrange(1, min(E, 12) + 1)
    T = int(2 ** rng.uniform(0, 16))
    return dict(T=max(1, min(T, 65535)), K=K, E=E, H=H, F=F, mapped=rng.choice([0, 1, E, rng.randrange(0, E + 1)]),
                waves=rng.choice([2, 2, 2, 1, 4, 8]), n_cus=rng.choice([256, 256, 304, 32]))


def check(p, c):
    """What launch_ffn and the kernels take for granted."""
    pairs, H, F = c["T"] * c["K"], c["H"], c["F"]
    assert p.pairs_cap == pairs and p.ksplit >= 1 and p.ksplit1 >= 1
    assert p.tiles_cap >= pairs // p.m_tile + min(c["E"], pairs)             # one partial tile for each expert at most
    if p.tiled:
        assert H % 64 == 0 and F % 64 == 0 and p.m_tile in (128, 256) and not p.halves
        assert p.ksplit <= F // 64 and p.ksplit1 <= H // 64
        if c["waves"] != 2:
            assert p.m_tile == 256 and p.ksplit1 == 1
        if c["waves"] in (4, 8):
            assert p.ksplit == 1
    else:
        assert p.m_tile == 128
        assert p.ksplit1 == 1 or p.ksplit1 * 64 <= H
    assert not p.g1_xcd or p.halves
    sizes = [("off_count", (c["E"] + 1) * 4), ("off_offset", (c["E"] + 2) * 4), ("off_sorted", pairs * 4), ("off_pos", pairs * 4),
             ("off_tile", p.tiles_cap * 16), ("off_ntiles", 8), ("off_h", max(pairs * F * 2, p.n_chunks * c["E"] * 4)),
             ("off_y", max(p.ksplit * pairs * H * 4, p.ksplit1 * pairs * 2 * F * 4 if p.ksplit1 > 1 else 0))]
    ends = [getattr(p, name) + size for name, size in sizes]
    starts = [getattr(p, name) for name, _ in sizes[1:]] + [p.bytes]
    assert all(a % 256 == 0 for a in starts) and all(e <= s for e, s in zip(ends, starts))
    assert p.n_chunks == (0 if pairs <= 14336 else -(-pairs // 4096))


def test_random_calls_at_any_buffer_size(rules):
    """The plan holds what the launcher requires; a buffer of the plan without splits is always enough, whatever is resident,
    and that plan asks for no more than a call of an unknown residency."""
    rng = random.Random(5)
    split = small = 0
    for _ in range(3000):
        c = random_call(rng)
        best, least = rules.plan(**c), rules.plain(**c)
        check(best, c)
        check(least, c)
        assert least.ksplit1 == 1 and not (least.tiled and least.m_tile == 128)
        assert least.bytes == rules.plain(**dict(c, mapped=0)).bytes
        for limit in (least.bytes, (least.bytes + best.bytes) // 2, best.bytes, least.bytes + rng.randrange(1 << 20)):
            if limit >= least.bytes:
                p = rules.plan(**c, limit=limit)
                check(p, c)
                assert p.bytes <= limit
        split += best.ksplit1 > 1
        small += best.tiled and best.m_tile == 128
    assert split > 300 and small > 50                                        # the draws reach the rules


def test_tiles_of_a_single_expert(rules):
    """128 x 128 tiles while 256 x 256 ones fill three quarters of the CUs at most: 4 * row tiles * column tiles <= 3 * 256."""
    of = lambda T, **kw: (lambda p: (bool(p.tiled), p.m_tile))(rules.plan(T=T, K=1, E=1, H=5120, F=1536, **kw))
    assert of(4096) == (True, 128) and of(4097) == (True, 256)               # 16 and 17 row tiles, 12 column tiles
    assert of(64) == (True, 128) and of(63) == (False, 128)                  # fewer rows: weight strips
    wide = lambda T, F: rules.plan(T=T, K=1, E=1, H=4096, F=F).m_tile        # up to 512 rows: a round and a half
    assert wide(512, 24576) == 128 and wide(512, 24640) == 256 and wide(513, 8192) == 128 and wide(513, 8256) == 256
    assert of(4096, waves=1) == (True, 256) and of(64, waves=8) == (False, 128)
    big = lambda T, F: rules.plan(T=T, K=1, E=1, H=5120, F=F).tiled          # strips again where the matrices are large
    assert big(64, 2176) and not big(64, 2240)                               # 6 H F on both sides of 64 MiB


def test_tiles_of_experts_that_are_resident(rules):
    """The rules look at the resident experts: waves of a quarter of 128 small experts, H 2048 F 512."""
    shape = dict(K=10, E=128, H=2048, F=512)
    of = lambda T, mapped, **kw: (lambda p: (bool(p.tiled), p.m_tile))(rules.plan(T=T, mapped=mapped, **dict(shape, **kw)))
    assert of(256, 32) == (True, 128) and of(256, 33) == (False, 128)        # 20 rows each, an eighth of the CUs
    assert of(256, 0) == (False, 128) and of(256, 128) == (False, 128)       # the whole layer fills the chip
    assert of(204, 32) == (False, 128)                   # 15.9 rows each
    assert of(256, 32, H=2112) == (False, 128)           # longer K: strips
    assert of(64, 32, E=32) == (False, 128) and of(64, 0, E=32) == (False, 128)        # no wave: every expert is resident
    assert of(64, 32, E=32, H=1024) == (True, 128) and of(64, 0, E=32, H=1088) == (False, 128)
    assert of(1638, 64) == (True, 256) and of(1638, 65) == (False, 128)      # 128 rows each: a second strip tile too often
    assert of(1638, 2) == (True, 256) and of(1638, 1) == (True, 128)         # one: small tiles
    assert of(1200, 32) == (True, 128)


def test_splits_of_the_first_product(rules):
    token = rules.plan(T=1, K=10, E=512, H=2048, F=512)
    assert not token.tiled and token.ksplit1 > 1         # 20 workgroups otherwise
    assert rules.plan(T=256, K=2, E=8, H=4096, F=14336).ksplit1 == 1         # 448
    ragged = rules.plan(T=333, K=4, E=64, H=2880, F=360)
    assert ragged.halves and ragged.g1_xcd and ragged.ksplit1 == 1           # three strips each, rows of 5.6 lines
    assert not rules.plan(T=333, K=4, E=64, H=2880, F=384).g1_xcd            # whole lines
    assert rules.plan(T=1, K=10, E=512, H=2048, F=512, waves=8).ksplit1 == token.ksplit1       # strips: no matter
    shared = rules.plan(T=512, K=1, E=1, H=5120, F=1536)
    assert shared.tiled and shared.ksplit1 > 1 and rules.plan(T=512, K=1, E=1, H=5120, F=1536, waves=8).ksplit1 == 1


def test_small_tiles_do_not_run_out_of_tile_numbers(rules):
    """The launcher takes 65535 row tiles at most, a call with more is refused: the choice of tiles never makes it so."""
    c = dict(T=65535, K=200, E=200, H=64, F=64)                              # 13.1 million pairs
    assert rules.plain(**c).tiles_cap <= 65535
    for mapped in (0, 1, 2, 200):
        p = rules.plan(**c, mapped=mapped)
        check(p, dict(c, waves=2))
        assert p.tiles_cap <= 65535
    rng = random.Random(6)
    for _ in range(2000):
        c = random_call(rng)
        c.update(T=rng.randrange(20000, 65536), K=rng.randrange(1, min(c["E"], 400) + 1))
        if rules.plain(**c).tiles_cap <= 65535:
            assert rules.plan(**c).tiles_cap <= 65535


def test_a_single_resident_expert_that_every_token_takes(rules):
    """128 x 128 tiles lose at many rows (H 5120 F 1536, 16384 rows: 921 us against 792).  With one of several experts resident
    its share of the pairs is not known; no token lists it twice, so T rows must still be few enough."""
    of = lambda T, E, mapped: rules.plan(T=T, K=2, E=E, H=5120, F=1536, mapped=mapped).m_tile
    assert of(16384, 8, 1) == 256 and of(4097, 8, 1) == 256 and of(4096, 8, 1) == 128


def test_splits_give_way_to_more_row_tiles_than_planned(rules):
    """Strips and 128 x 128 tiles: split while the tiles leave CUs without work, or as many as the plan expected."""
    p = rules.plan(T=1024, K=8, E=160, H=5120, F=1536, mapped=4)             # 51 rows each planned, 1024 if all take these
    assert p.halves and p.ksplit1 > 1 and p.split_tiles == 255 // 12
    p = rules.plan(T=1024, K=10, E=128, H=2048, F=512, mapped=8)
    assert p.tiled and p.m_tile == 128 and p.ksplit1 > 1 and p.split_tiles == 255 // 8
    p = rules.plan(T=256, K=2, E=8, H=4096, F=14336)
    assert p.ksplit1 == 1 and p.split_tiles == 0
    # 256 x 256 tiles: a plan that the model shares is kept, and past it the model decides
    p = rules.plan(T=512, K=2, E=8, H=4096, F=1792)
    assert p.tiled and p.m_tile == 256 and (p.ksplit1, p.split_tiles) == (2, 8)
    assert rules.least_cost(4096, 1792, 256, 8, 1024, 2) == 2                # 4 pairs of (super-tile, split) on each of 8 XCDs' 32 CUs
    assert rules.least_cost(4096, 1792, 256, 9, 1024, 2) == 1                # 12 pairs: a second round on four of them
    p = rules.plan(T=1024, K=8, E=20, H=5120, F=384)
    assert p.ksplit1 == 2 and p.split_tiles == 0 and rules.least_cost(5120, 384, 256, 40, 8192, 2) == 1
    assert rules.least_cost(5120, 384, 256, 20, 3200, 4) > 1
    for n_tiles in (0, 1, 3, 4, 5, 1000, 65535):                             # any count is a valid question
        assert 1 <= rules.least_cost(64, 64, 256, n_tiles, n_tiles * 256, 8) <= 8
    assert rules.least_cost(4096, 1792, 4, 8, 1024, 2) in (1, 2)             # fewer CUs than XCDs
