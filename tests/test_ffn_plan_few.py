"""The launch plan of calls of up to 64 pairs (csrc/ffn_plan.h), compiled on its own."""
import ctypes as C
import os
import random
import subprocess
from types import SimpleNamespace

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")
FIELDS = ("few", "few_fused", "few_splits", "halves", "ksplit", "ksplit1", "bytes", "off_y", "off_part", "tiled")
SHIM = """
#include "ffn_plan.h"
using namespace fluxmoe;
extern "C" void plan(uint64_t E, uint64_t H, uint64_t F, uint32_t T, uint32_t K, uint64_t limit, uint32_t mapped, uint64_t* o) {
    const FfnPlan p = plan_ffn(FfnShape{E, H, F, 256, 2, true}, T, K, limit, mapped); %s
}
extern "C" void general(uint64_t E, uint64_t H, uint64_t F, uint32_t T, uint32_t K, uint64_t limit, uint32_t mapped, uint64_t* o) {
    const FfnPlan p = plan_ffn(FfnShape{E, H, F, 256, 2, true, false}, T, K, limit, mapped); %s
}
extern "C" uint64_t asked(uint64_t E, uint64_t H, uint64_t F, uint32_t T, uint32_t K) { return ffn_bytes(FfnShape{E, H, F, 256, 2, true}, T, K); }
extern "C" uint64_t quarter(uint64_t F, uint64_t k) { return few_quarter(F, k); }
""" % ((" ".join("o[%d] = p.%s;" % (i, f) for i, f in enumerate(FIELDS)),) * 2)


@pytest.fixture(scope="module")
def few(tmp_path_factory):
    d = tmp_path_factory.mktemp("ffn_plan_few")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    so = C.CDLL(str(d / "shim.so"))
    so.plan.argtypes = so.general.argtypes = [C.c_uint64] * 3 + [C.c_uint32] * 2 + [C.c_uint64, C.c_uint32, C.POINTER(C.c_uint64)]
    so.asked.argtypes, so.asked.restype = [C.c_uint64] * 3 + [C.c_uint32] * 2, C.c_uint64
    so.quarter.argtypes, so.quarter.restype = [C.c_uint64] * 2, C.c_uint64

    def call(fn):
        def plan(T, K, E, H, F, mapped=0, limit=2 ** 64 - 1):
            o = (C.c_uint64 * len(FIELDS))()
            fn(E, H, F, T, K, limit, mapped, o)
            return SimpleNamespace(**dict(zip(FIELDS, o)))
        return plan
    return SimpleNamespace(plan=call(so.plan), general=call(so.general), asked=so.asked, quarter=so.quarter)


def k_per(k, splits, unit):
    return min(k, -(-(-(-k // splits)) // unit) * unit)


def chains(few, p, H, F):
    """k rows that the first and the second product add up in one accumulator"""
    return (k_per(H, p.ksplit1, 256 if p.halves else 128) // (2 if p.halves else 1),
            min(F, few.quarter(F, p.few_splits)) if p.few_splits else k_per(F, p.ksplit, 32))


def random_call(rng):
    E = rng.choice([1, 2, 8, 20, 64, 160, 512])
    K = rng.randrange(1, min(E, 16) + 1)
    return dict(T=rng.randrange(1, 64 // K + 1), K=K, E=E, H=8 * rng.randrange(1, 700), F=8 * rng.randrange(1, rng.choice([80, 300, 1800])))


def test_random_calls_at_any_buffer_size(few, monkeypatch):
    """The scratch covers what the kernels write, sums that the second product adds up itself lie behind its own, its K splits have
    work, and shorter buffers are given way to."""
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)
    rng = random.Random(7)
    seen = {"fused": 0, "few": 0, "split": 0, "old": 0}
    for _ in range(3000):
        E = rng.choice([1, 2, 8, 20, 64, 160, 512])
        K = rng.randrange(1, min(E, 16) + 1)
        T = rng.randrange(1, 64 // K + 1)
        H, F = 8 * rng.randrange(1, 700), 8 * rng.randrange(1, rng.choice([20, 80, 1000]))
        mapped = rng.choice([0, E, max(1, E // 2)])
        c = dict(T=T, K=K, E=E, H=H, F=F, mapped=mapped)
        best = few.plan(**c)
        for limit in (2 ** 64 - 1, best.bytes - 1, best.off_y + T * K * H * 4 + 255, rng.randrange(best.off_y, best.bytes + 1)):
            p = few.plan(**c, limit=limit)
            if p.tiled:
                continue
            pairs = T * K
            assert p.few and (p.bytes <= limit or p.ksplit1 == 1)
            y = (p.few_splits or p.ksplit) * pairs * H * 4
            part = p.ksplit1 * pairs * 2 * F * 4 if p.ksplit1 > 1 else 0
            assert p.bytes >= p.off_y + y and p.bytes >= p.off_part + part and p.off_part % 256 == 0
            assert p.off_part == p.off_y or (p.few_fused and p.off_part >= p.off_y + y)
            assert p.ksplit1 <= max(1, H // 64)
            if p.few_fused:
                assert p.few_splits and p.ksplit1 > 1 and T <= 4 and few.quarter(F, p.few_splits) <= 256
            if p.few_splits > 1:
                assert (p.few_splits - 1) * 256 < F
            seen["fused" if p.few_fused else "split" if p.few_splits > 1 else "few" if p.few_splits else "old"] += 1
        if not best.tiled and mapped in (0, E):
            assert few.asked(E, H, F, T, K) >= few.plan(**dict(c, mapped=0)).bytes
    assert all(v > 100 for v in seen.values()), seen


def test_both_sides_of_the_lines(few):
    of = lambda **kw: few.plan(**kw)
    token = dict(K=10, E=512, H=2048, F=512)
    assert of(T=1, **token).few_fused and of(T=1, **dict(token, F=1024)).few_fused and not of(T=1, **dict(token, F=1032)).few_fused
    wide = dict(T=1, K=8, E=160, H=5120)                                     # 320 workgroups
    assert of(F=512, **wide).few_fused and not of(F=520, **wide).few_fused
    assert of(T=4, K=2, E=64, H=2048, F=512).few_fused and not of(T=5, K=2, E=64, H=2048, F=512).few_fused
    assert of(T=6, K=10, E=512, H=2048, F=512).few_splits == 0               # 16 strips of about 57 experts
    assert of(T=1, K=1, E=8, H=4096, F=14336).few_splits == 8                # 32 strips of one
    assert of(T=1, K=8, E=8, H=4096, F=14336).few_splits == 0                # quarters of 3584 k
    assert of(T=7, K=10, E=512, H=2048, F=512).few == 0                      # 70 pairs
    five = dict(T=9, K=5, E=8, H=2232)                                       # 144 workgroups, no second round of them
    assert [of(F=F, **five).few_splits for F in (432, 864, 1024, 1280, 1728, 2048)] == [1, 1, 1, 0, 0, 0]
    assert of(T=59, K=1, E=4, H=4752, F=1680).few_splits == 0 and of(T=11, K=4, E=4, H=4768, F=3736).few_splits == 0


def test_a_round_of_whole_strips_keeps_the_general_first_product(few, monkeypatch):
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)
    for E, H, F, T, K in [(32, 1080, 6360, 5, 8), (64, 2560, 2176, 10, 4), (42, 2960, 9336, 10, 4), (32, 3480, 3200, 6, 10), (20, 992, 3552, 10, 6)]:
        p, g = (f(E=E, H=H, F=F, T=T, K=K) for f in (few.plan, few.general))
        assert p.few and (p.ksplit1, p.halves) == (g.ksplit1, g.halves)
    # tiles of more than 16 rows are unlikely, or not
    few_rows = dict(E=4, H=512, F=256)
    assert [few.plan(T=T, K=2, **few_rows).few_splits > 0 for T in (16, 20, 26, 32)] == [True, True, False, False]
    assert few.plan(T=15, K=4, **few_rows).few_splits and few.plan(T=40, K=1, E=8, H=512, F=256).few_splits
    skewed = dict(H=512, F=256, E=16)                                        # 0.3 of the tokens for each of their experts
    assert [few.plan(T=T, K=K, **skewed).few_splits > 0 for T, K in ((53, 1), (54, 1), (26, 2), (27, 2), (17, 3), (18, 3))] == [True, False] * 3
    rng, halved = random.Random(12), 0
    for c in (random_call(rng) for _ in range(8000)):
        c["F"] = c["F"] // 256 * 256 or 256                                  # an even number of strips
        p = few.plan(**c, mapped=c["E"])
        if p.few and c["T"] == 1:                                            # K row tiles
            assert not p.halves or c["F"] // 256 * c["K"] < 256, c
            halved += p.halves
    assert halved > 20


def test_more_experts_a_token_than_the_layer_has(tmp_path):
    """The size query takes any number of experts a token: no conversion of a number that is none."""
    (tmp_path / "m.cpp").write_text("""
#include "ffn_plan.h"
int main() {
    for (uint64_t E = 1; E <= 4; ++E)
        for (uint32_t T = 1; T <= 8; ++T)
            for (uint32_t K = 1; T * K <= 64; ++K) fluxmoe::ffn_bytes(fluxmoe::FfnShape{E, 512, 512, 256, 2, true}, T, K);
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=float-cast-overflow", "-fsanitize-undefined-trap-on-error", "-I", CSRC, str(tmp_path / "m.cpp"),
                    "-o", str(tmp_path / "m")], check=True)
    subprocess.run([str(tmp_path / "m")], check=True)


def test_no_sum_is_longer_than_in_the_general_kernels(few, monkeypatch):
    """Against the plan of a call that is not routed, which has the same rules without those for few pairs."""
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)
    rng = random.Random(8)
    calls = [dict(E=8, H=2176, F=1736, T=8, K=7), dict(E=20, H=2480, F=1904, T=1, K=10), dict(E=4, H=4280, F=1816, T=22, K=2)]
    seen = 0
    for c in calls + [random_call(rng) for _ in range(20000)]:
        mapped = rng.randrange(c["E"] + 1)
        p, g = few.plan(**c, mapped=mapped), few.general(**c, mapped=mapped)
        if p.few:
            a, b = chains(few, p, c["H"], c["F"]), chains(few, g, c["H"], c["F"])
            assert a[0] <= b[0] and a[1] <= b[1], (c, mapped)
            seen += p.few_splits > 0 and p.few_splits != g.ksplit
    assert seen > 1000


def test_short_buffers_keep_the_sums_short(few, monkeypatch):
    """In any buffer that holds the general plan: no sum longer than in it, and no quarter past the rule's line."""
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)
    rng = random.Random(9)
    calls = [dict(E=8, H=4096, F=14336, T=1, K=1), dict(E=8, H=4928, F=9552, T=1, K=2), dict(E=512, H=2048, F=512, T=1, K=10)]
    gave = 0
    for c in calls + [random_call(rng) for _ in range(8000)]:
        mapped = rng.randrange(c["E"] + 1)
        best = few.plan(**c, mapped=mapped)
        for limit in (best.bytes - 1, rng.randrange(best.off_y, best.bytes + 1)):
            p, g = few.plan(**c, mapped=mapped, limit=limit), few.general(**c, mapped=mapped, limit=limit)
            assert (p.bytes <= limit) == (g.bytes <= limit)
            if p.few and p.bytes <= limit:
                a, b = chains(few, p, c["H"], c["F"]), chains(few, g, c["H"], c["F"])
                assert a[0] <= b[0] and a[1] <= b[1], (c, mapped, limit)
                assert p.few_fused or not p.few_splits or few.quarter(c["F"], p.few_splits) <= 1024
                gave += (p.few_splits, p.few_fused, p.ksplit1) != (best.few_splits, best.few_fused, best.ksplit1)
    assert gave > 1000
    # the first product's sums are what does not fit: the second product keeps its splits
    whole = few.plan(**calls[0])
    short = few.plan(**calls[0], limit=whole.bytes - 1)
    assert whole.few_splits == short.few_splits == 8 and short.ksplit1 < whole.ksplit1


def test_the_query_covers_every_number_of_resident_experts(few, monkeypatch):
    """A wave of any part of the layer takes the plan it would take without a limit in a buffer of the size asked for."""
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)
    rng = random.Random(10)
    calls = [(dict(E=16, H=2048, F=12728, T=7, K=7), 6), (dict(E=8, H=1952, F=10232, T=6, K=8), 7), (dict(E=8, H=4928, F=9552, T=1, K=2), 6)]
    calls += [(c, rng.randrange(1, c["E"] + 1)) for c in (random_call(rng) for _ in range(3000))]
    for c, mapped in calls:
        best, p = few.plan(**c, mapped=mapped), few.plan(**c, mapped=mapped, limit=few.asked(c["E"], c["H"], c["F"], c["T"], c["K"]))
        assert vars(p) == vars(best), (c, mapped)


def test_the_plan_report_tells_the_splits_that_run(few, monkeypatch):
    from paper_2604_02715_amd import binding as B
    monkeypatch.delenv("FLUXMOE_FFN_MTILE", raising=False)
    rng = random.Random(11)
    other = 0
    for c in [dict(E=512, H=2048, F=512, T=1, K=10)] + [random_call(rng) for _ in range(200)]:
        ctx = B.fluxmoe_create(1, c["E"], c["H"], c["F"], c["E"])
        try:
            said = B.fluxmoe_ffn_plan(ctx, c["T"], c["K"])
        finally:
            B.fluxmoe_destroy(ctx)
        p, g = few.plan(**c, mapped=c["E"]), few.general(**c, mapped=c["E"])
        if p.few:
            assert said == (128, p.few_splits or g.ksplit)
            other += said[1] != g.ksplit
    assert other > 20
