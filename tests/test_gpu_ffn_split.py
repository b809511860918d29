"""GPU parity of the expert FFN where the first product is split over K (few workgroups otherwise: a token or two,
a single expert, narrow ffn) and of the shared expert's own grouping, against the FP64 oracle.  Tolerance as in
test_gpu_ffn.py: the sums stay FP32, only their order changes."""
import numpy as np
import pytest
import torch

from oracle import ffn as offn
from oracle import paging
from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import inputs
from test_ffn_plan import rules  # noqa: F401 (fixture)
from test_ffn_plan_ragged import plan  # noqa: F401 (fixture)
from test_gpu_ffn import TOL, run_ffn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(tokens=1, top_k=2, hidden=1032, ffn=136),                              # split at 128 k, a last split with a k tail
    dict(tokens=5, top_k=3, hidden=2056, ffn=72),                               # one strip, partly empty
    dict(tokens=100, top_k=1, n_experts=1, n_slots=1, hidden=2048, ffn=200),    # one expert, 100 rows in one tile
    dict(tokens=40, top_k=2, hidden=1024, ffn=264, routing="zipf"),
    dict(tokens=300, top_k=1, n_experts=1, n_slots=1, hidden=1024, ffn=192),    # LDS-tiled kernels, ragged column tile
    dict(tokens=700, top_k=2, n_experts=3, n_slots=3, hidden=1600, ffn=320),    # the same, splits of unequal length
])
def test_split_first_product(kw):
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw), seed=8)


def test_split_first_product_in_waves():
    """Half of the experts resident at a time: pairs of the others are skipped and the sums are only made for the rest."""
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=20, top_k=3, hidden=1024, ffn=136, n_slots=4)
    run_ffn_case(cfg, seed=9, waves=lambda u: paging.waves(u, 4))


@pytest.mark.parametrize("tokens", [1, 100, 129, 257, 600])
@pytest.mark.parametrize("shape", [(1024, 192), (1096, 200)])
def test_shared_expert(tokens, shape):
    """Row tiles of one, several and partly filled, whole steps and tails (gemm_ring_kernel)."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=2, shared_expert=True, tokens=tokens, hidden=shape[0], ffn=shape[1])
    pool, _ = build_pool(cfg)
    try:
        s13, s2 = inputs.shared_expert_weights(cfg, 0)
        x = inputs.activations(cfg)
        s13d, s2d, xd = s13.cuda(), s2.cuda(), x.cuda()
        out = torch.full((tokens, cfg.hidden), 5.0, dtype=torch.float32, device="cuda")
        pool.shared_expert_ffn(s13d, s2d, xd, out)
        once = out.clone()
        pool.shared_expert_ffn(s13d, s2d, xd, out, B.FFN_ACCUMULATE)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
        want = offn.moe_ffn(inputs.bits_u16(x), np.zeros((tokens, 1), dtype=np.int32), np.ones((tokens, 1), dtype=np.float32),
                            lambda e: (inputs.bits_u16(s13), inputs.bits_u16(s2)))
        assert offn.rel_frobenius(once.cpu().numpy(), want) <= TOL
        assert torch.equal(out, once + once)
    finally:
        pool.close()


@pytest.mark.parametrize("kw", [
    dict(tokens=64, top_k=1, n_experts=1, n_slots=1, hidden=512, ffn=64),       # one tile of 128 x 128, gate and up 64 columns each
    dict(tokens=129, top_k=1, n_experts=1, n_slots=1, hidden=1088, ffn=576),    # second row tile of one row, ragged column tiles, splits
    dict(tokens=600, top_k=1, n_experts=1, n_slots=1, hidden=64, ffn=128),      # one and two k steps
    dict(tokens=100, top_k=4, n_experts=6, n_slots=6, hidden=320, ffn=192),     # several experts
    dict(tokens=150, top_k=5, n_experts=30, n_slots=30, hidden=1024, ffn=256, routing="zipf"),   # row tiles from 1 to 128 rows
    dict(tokens=400, top_k=2, n_experts=6, n_slots=6, hidden=1024, ffn=512),    # 133 rows each on few strips: tiles of 256
])
def test_tiles_of_launches_with_few_strips(kw):
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw), seed=10)


@pytest.mark.parametrize("kw,refused_below", [
    (dict(tokens=3, top_k=2, hidden=1024, ffn=512), True),                                      # strips, four splits
    (dict(tokens=300, top_k=1, n_experts=1, n_slots=1, hidden=2048, ffn=1024), False),          # tiles of 128, both products split
    (dict(tokens=600, top_k=2, n_experts=4, n_slots=4, hidden=2048, ffn=512), True),            # tiles of 256, four splits
])
def test_a_buffer_for_the_plan_without_splits_is_enough(kw, refused_below, rules):
    """A call prefers a plan that takes more scratch than the one without K splits of the first product; a buffer of that
    plan's size must do, as must one in between, and give the same result to rounding.  One byte less is refused, except
    where the small tiles need less still."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw)
    call = dict(T=cfg.tokens, K=cfg.top_k, E=cfg.n_experts, H=cfg.hidden, F=cfg.ffn, mapped=cfg.n_experts)
    best, least = rules.plan(**call), rules.plain(**call)
    assert best.ksplit1 > rules.plan(**call, limit=least.bytes).ksplit1 and least.bytes < best.bytes
    pool, dense = build_pool(cfg)
    try:
        assert pool.ws_bytes - int(pool.sizes.pool_workspace_bytes) >= best.bytes
        x = inputs.activations(cfg).cuda()
        ids, g = inputs.routing(cfg)
        idd, gd = torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda()
        pool.reset_page_table()
        every = np.arange(cfg.n_experts)
        pool.materialize(0, every, every)
        bind = lambda scratch: B.fluxmoe_bind_arenas(pool.ctx, pool.slots13.data_ptr(), pool.slots2.data_ptr(), pool.workspace.data_ptr(),
                                                     int(pool.sizes.pool_workspace_bytes) + scratch)
        outs = []
        for scratch in (best.bytes, (best.bytes + least.bytes) // 2, least.bytes):
            bind(scratch)
            pool.workspace[int(pool.sizes.pool_workspace_bytes):].fill_(0x7F)
            out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
            pool.expert_ffn(0, x, idd, gd, out)
            torch.cuda.synchronize()
            assert (pool.workspace[int(pool.sizes.pool_workspace_bytes) + scratch:] == 0x7F).all()
            outs.append(out.cpu().numpy())
        assert pool.device_errors() == 0
        want = offn.moe_ffn(inputs.bits_u16(x.cpu()), ids, g, lambda e: (inputs.bits_u16(dense[0][0][e]), inputs.bits_u16(dense[0][1][e])))
        for out in outs:
            assert offn.rel_frobenius(out, want) <= TOL
        bind(least.bytes - 1 if refused_below else least.bytes // 4)
        with pytest.raises(B.FluxmoeError) as ei:
            pool.expert_ffn(0, x, idd, gd, torch.zeros((cfg.tokens, cfg.hidden), device="cuda"))
        assert ei.value.status == -2
    finally:
        pool.close()


@pytest.mark.parametrize("kw", [
    dict(tokens=1, top_k=1),
    dict(tokens=32, top_k=2),                                                    # 64 pairs, the most that are grouped this way
    dict(tokens=64, top_k=1, n_experts=2, n_slots=2, hidden=136, ffn=264),       # tiles of 17 to 64 rows, ragged edges
    dict(tokens=13, top_k=5, n_experts=300, n_slots=300, hidden=64, ffn=72),     # one more pair: the grouping kernel
    dict(tokens=6, top_k=10, n_experts=200, n_slots=200, hidden=520, ffn=72, routing="uniform"),
])
def test_few_pairs(kw):
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw), seed=11)


def test_few_pairs_on_one_expert_on_absent_ones_and_on_ids_out_of_range():
    """Grouping by the first product's own workgroups: every pair on one expert; half of the experts absent, skipped or
    flagged; ids out of range are flagged and add nothing."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=20, top_k=3)
    run_ffn_case(inputs.scaled(cfg, tokens=60, top_k=1), seed=12, ids_override=lambda ids: np.full_like(ids, 5))
    run_ffn_case(cfg, seed=13, waves=lambda u: paging.waves(u, 4))
    pool, dense = build_pool(cfg)
    try:
        w13, w2 = dense[0]
        x = inputs.activations(cfg)
        ids, g = inputs.routing(cfg)
        ids[3, 1], ids[7, 0], ids[19, 2] = -1, 8, 2 ** 31 - 1
        pool.reset_page_table()
        pool.materialize(0, np.arange(8), np.arange(8))
        out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
        gd = torch.from_numpy(g).cuda()
        pool.expert_ffn(0, x.cuda(), torch.from_numpy(ids).cuda(), gd, out, B.FFN_SKIP_UNMAPPED)
        torch.cuda.synchronize()
        assert pool.device_errors() == 2                     # skipping covers absent experts, not bad ids
        bad = (ids < 0) | (ids >= 8)
        kept, good_ids = np.where(bad, 0, g).astype(np.float32), ids.copy()
        for t, k in np.argwhere(bad):                        # an expert the token does not list, with gate 0
            good_ids[t, k] = next(e for e in range(8) if e not in ids[t])
        want = offn.moe_ffn(inputs.bits_u16(x), good_ids, kept, lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
        assert offn.rel_frobenius(out.cpu().numpy(), want) <= TOL
        pool.release(0, [0, 1, 2, 3])
        good = torch.from_numpy(good_ids).cuda()
        pool.expert_ffn(0, x.cuda(), good, gd, out)
        torch.cuda.synchronize()
        assert pool.device_errors() == 2
        pool.expert_ffn(0, x.cuda(), good, gd, out, B.FFN_SKIP_UNMAPPED)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
    finally:
        pool.close()


@pytest.mark.parametrize("kw", [
    dict(tokens=100, top_k=2, hidden=264, ffn=64),                               # one strip, one pair of k blocks and a tail of 8
    dict(tokens=100, top_k=2, hidden=392, ffn=360, n_experts=3, n_slots=3),      # three strips, a block and a tail left over
    dict(tokens=90, top_k=4, hidden=1288, ffn=136, n_experts=20, n_slots=20, routing="zipf"),   # tiles of every size, ragged strip
    dict(tokens=100, top_k=2, hidden=120, ffn=72),                               # less than a block of k
    dict(tokens=2, top_k=4, hidden=1544, ffn=264),                               # grouped by its own workgroups
])
def test_halves_of_k_in_one_workgroup(kw):
    """Few or an odd number of strips: the two pairs of wavefronts of a workgroup share a strip and halve its k range."""
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw), seed=14)


@pytest.mark.parametrize("kw", [
    dict(tokens=7168, top_k=2, hidden=64, ffn=128),                              # 14336 pairs: the most one workgroup groups
    dict(tokens=7169, top_k=2, hidden=64, ffn=64, n_experts=40, n_slots=40, routing="zipf"),    # several, the last chunk short
])
def test_edges_of_the_grouping_by_several_workgroups(kw):
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw), seed=15)


@pytest.mark.parametrize("shape", [(2048, 64, 2), (1856, 192, 5)])
def test_walking_second_product(shape):
    """Short K and more 256 x 256 tiles of the second product than workgroups: a workgroup takes several, ragged last
    column tile and row tiles with few rows among them."""
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=9000, top_k=1, n_experts=shape[2], n_slots=shape[2], hidden=shape[0], ffn=shape[1])
    run_ffn_case(cfg, seed=16)


@pytest.mark.parametrize("kw", [
    dict(tokens=2000, top_k=2, n_experts=64, hidden=1024, ffn=2056),             # strips: 32 row tiles where one or two were planned
    dict(tokens=300, top_k=2, n_experts=64, hidden=1024, ffn=2056),              # few enough to split as planned
    dict(tokens=5000, top_k=1, n_experts=64, hidden=2048, ffn=1024),             # tiles of 128 x 128: 40 where one was planned
    dict(tokens=1200, top_k=2, n_experts=8, hidden=2048, ffn=512),               # tiles of 256 x 256: four splits,
    dict(tokens=3000, top_k=2, n_experts=8, hidden=2048, ffn=512),               # two of the four that were planned,
    dict(tokens=6000, top_k=2, n_experts=8, hidden=2048, ffn=512),               # one
])
def test_every_token_on_the_resident_experts(kw):
    """The plan counts on the resident experts' mean share of the pairs; here they get all of them, and the kernels, which
    see the row tiles, decide how many splits of the first product work."""
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_slots=2, **kw)
    run_ffn_case(cfg, seed=17, ids_override=lambda ids: np.broadcast_to(np.arange(ids.shape[1], dtype=np.int32), ids.shape).copy())


@pytest.mark.parametrize("rows", [1, 32, 33, 64, 65, 97, 128, 129, 160, 193, 225, 256, 289])
def test_row_groups_of_the_lds_tiled_kernels(rows, monkeypatch):
    """Tiles of 256 x 256 with every number of 32-row groups: the wavefronts' groups beyond the tile's rows are not
    fetched or multiplied."""
    monkeypatch.setenv("FLUXMOE_FFN_MTILE", "256")
    run_ffn_case(inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=rows, top_k=1, n_experts=1, n_slots=1, hidden=256, ffn=192), seed=3)


@pytest.mark.parametrize("kw", [
    dict(tokens=300, top_k=1, n_experts=1, n_slots=1, hidden=8, ffn=40),        # a partial step is all there is
    dict(tokens=700, top_k=2, n_experts=3, n_slots=3, hidden=200, ffn=328),     # tails of 8 in both products, ragged columns
    dict(tokens=300, top_k=1, n_experts=2, n_slots=2, hidden=264, ffn=2056),
    dict(tokens=2600, top_k=2, n_experts=20, n_slots=20, hidden=136, ffn=72),
    dict(tokens=520, top_k=1, n_experts=2, n_slots=2, hidden=256, ffn=1032),    # one product whole, one with a partial step
])
def test_strips_where_tiles_would_be_taken_for_longer_k(kw, plan):
    """Rows enough for 256 x 256 tiles, K too short for the splits that would stand for the strips' halves."""
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw)
    assert not plan(cfg.tokens, cfg.top_k, cfg.n_experts, cfg.hidden, cfg.ffn, mapped=cfg.n_experts).tiled
    run_ffn_case(cfg, seed=12)


def ragged_cfg(T, K, E, H, F):
    return inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=T, top_k=K, n_experts=E, n_slots=E, hidden=H, ffn=F)


@pytest.mark.parametrize("call,ksplit1,ksplit", [
    ((600, 2, 4, 1096, 1000), 2, 3),            # splits that stand for the strips' halves
    ((143, 1, 1, 792, 728), 2, 2),              # both products split, the last split of each with a partial step
    ((383, 1, 2, 776, 136), 2, 1),              # the second walks
    ((889, 3, 6, 8, 1544), 1, 6),               # a partial step is all of the first product's k
    ((5532, 2, 6, 8, 272), 1, 1),               # several tiles for a workgroup, row tiles of every size
    ((874, 3, 20, 688, 1656), 1, 6),            # non-temporal weights: first product unsplit, second split
    ((1856, 3, 30, 1032, 760), 1, 1),           # and both unsplit
])
def test_large_tiles_with_a_partial_step(call, ksplit1, ksplit, plan):
    cfg = ragged_cfg(*call)
    ctx = B.fluxmoe_create(1, cfg.n_experts, cfg.hidden, cfg.ffn, cfg.n_slots)
    limit = B.fluxmoe_ffn_workspace_bytes(ctx, cfg.tokens, cfg.top_k)
    B.fluxmoe_destroy(ctx)
    p = plan(*call, mapped=cfg.n_experts, limit=limit)
    assert (p.tiled, p.m_tile, p.ksplit1, p.ksplit) == (1, 256, ksplit1, ksplit)
    run_ffn_case(cfg, seed=12)


@pytest.mark.parametrize("call", [(600, 2, 4, 1096, 1000), (881, 8, 8, 928, 392)])
def test_ragged_shapes_in_smaller_buffers_and_in_the_static_scratch(call, plan):
    """Tiles with their splits, the strips' plan in its own bytes, the plan without splits, and what 32 MiB hold."""
    from gpu_common import build_pool
    cfg = ragged_cfg(*call)
    every = np.arange(cfg.n_experts)
    of = lambda **kw: plan(*call, mapped=cfg.n_experts, **kw)
    best, strips, least = of(), of(ragged=False), of(split=False)
    assert best.tiled and best.bytes > strips.bytes >= least.bytes and of(limit=strips.bytes).__dict__ == strips.__dict__ and strips.halves
    assert bool(of(limit=32 << 20).tiled) == (best.bytes <= 32 << 20)
    pool, dense = build_pool(cfg)
    try:
        pool_bytes = int(pool.sizes.pool_workspace_bytes)
        assert pool.ws_bytes - pool_bytes >= best.bytes
        x = inputs.activations(cfg).cuda()
        ids, g = inputs.routing(cfg)
        idd, gd = torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda()
        pool.reset_page_table()
        pool.materialize(0, every, every)
        want = offn.moe_ffn(inputs.bits_u16(x.cpu()), ids, g, lambda e: (inputs.bits_u16(dense[0][0][e]), inputs.bits_u16(dense[0][1][e])))
        for scratch in (best.bytes, (best.bytes + strips.bytes) // 2, strips.bytes, least.bytes):
            B.fluxmoe_bind_arenas(pool.ctx, pool.slots13.data_ptr(), pool.slots2.data_ptr(), pool.workspace.data_ptr(), pool_bytes + scratch)
            pool.workspace[pool_bytes:].fill_(0x7F)
            out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
            pool.expert_ffn(0, x, idd, gd, out)
            torch.cuda.synchronize()
            assert (pool.workspace[pool_bytes + scratch:] == 0x7F).all()
            assert offn.rel_frobenius(out.cpu().numpy(), want) <= TOL
        out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
        B.fluxmoe_expert_ffn_static(pool.ctx, 0, x.data_ptr(), cfg.tokens, idd.data_ptr(), gd.data_ptr(), cfg.top_k, pool.page_table.data_ptr(), out.data_ptr(), 0,
                                    torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0 and offn.rel_frobenius(out.cpu().numpy(), want) <= TOL
    finally:
        pool.close()


def test_what_lies_behind_the_operands_stays_out_of_the_tiles(plan):
    """The pieces past the end of K are zeros: the slot behind the routed expert's and one token are infinite here, which makes that
    token's row infinite or not a number, and no other."""
    from gpu_common import build_pool
    cfg = ragged_cfg(143, 1, 1, 792, 728)
    cfg = inputs.scaled(cfg, n_slots=2)
    p = plan(143, 1, 1, 792, 728, mapped=1)
    assert p.tiled and p.ksplit1 == 2 and p.ksplit == 2
    pool, dense = build_pool(cfg)
    try:
        w13, w2 = dense[0]
        x, (ids, g) = inputs.activations(cfg).clone(), inputs.routing(cfg)
        x[100] = float("inf")
        out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
        pool.poison_slots(0x7F80)
        pool.reset_page_table()
        pool.materialize(0, np.arange(1, dtype=np.int32), np.arange(1, dtype=np.int32))
        pool.expert_ffn(0, x.cuda(), torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda(), out)
        torch.cuda.synchronize()
        assert bool(torch.isinf(pool.slot2(1).view(torch.bfloat16)).all())
        others = [t for t in range(cfg.tokens) if t != 100]
        assert not bool(torch.isfinite(out[100]).any())
        want = offn.moe_ffn(inputs.bits_u16(x[others].contiguous()), ids[others], g[others], lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
        assert offn.rel_frobenius(out[others].cpu().numpy(), want) <= TOL
    finally:
        pool.close()


def test_infinite_weights_past_whole_steps_stay_where_they_belong(plan):
    """An infinite weight in the last k row of the second product reaches its own column only."""
    from gpu_common import build_pool
    cfg = ragged_cfg(143, 1, 1, 792, 728)
    assert plan(143, 1, 1, 792, 728, mapped=1).tiled
    pool, dense = build_pool(cfg)
    try:
        x, (ids, g) = inputs.activations(cfg), inputs.routing(cfg)
        out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
        pool.reset_page_table()
        pool.materialize(0, np.arange(1, dtype=np.int32), np.arange(1, dtype=np.int32))
        torch.cuda.synchronize()
        pool.slot2(0).view(torch.bfloat16).view(cfg.ffn, cfg.hidden)[cfg.ffn - 1, 5] = float("inf")
        pool.expert_ffn(0, x.cuda(), torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda(), out)
        torch.cuda.synchronize()
        bad = ~torch.isfinite(out.cpu())
        assert bool(bad[:, 5].all()) and int(bad.sum()) == cfg.tokens
    finally:
        pool.close()


@pytest.mark.parametrize("tokens", [8191, 8193])
def test_sums_on_both_sides_of_the_memory_side_cache(tokens):
    """268.4 MB of partial sums (8192 tokens, top-1 of 2, H 8192): just below and above, with and without accumulation."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=tokens, top_k=1, n_experts=2, n_slots=2, hidden=8192, ffn=64)
    pool, dense = build_pool(cfg, gen_device="cuda")
    try:
        w13, w2 = dense[0]
        x, (ids, g) = inputs.activations(cfg), inputs.routing(cfg)
        out = torch.full((tokens, cfg.hidden), 5.0, dtype=torch.float32, device="cuda")
        pool.reset_page_table()
        pool.materialize(0, np.arange(2, dtype=np.int32), np.arange(2, dtype=np.int32))
        args = (0, x.cuda(), torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda(), out)
        pool.expert_ffn(*args)
        once = out.clone()
        pool.expert_ffn(*args, flags=B.FFN_ACCUMULATE)
        torch.cuda.synchronize()
        assert torch.equal(out, once + once)
        some = np.r_[0:64, tokens - 64:tokens]
        want = offn.moe_ffn(inputs.bits_u16(x[some].contiguous()), ids[some], g[some], lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
        assert offn.rel_frobenius(once[torch.from_numpy(some).cuda()].cpu().numpy(), want) <= TOL
    finally:
        pool.close()


@pytest.mark.parametrize("resident", [1, 3])
def test_sums_of_a_wave_on_both_sides_of_the_memory_side_cache(resident):
    """12000 tokens, top-1 of 4, H 8192: 393 MB if every pair is there, 98 MB of one expert's, 295 MB of three's; overwritten and
    accumulated."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=12000, top_k=1, n_experts=4, n_slots=4, hidden=8192, ffn=64)
    pool, dense = build_pool(cfg, gen_device="cuda")
    try:
        w13, w2 = dense[0]
        x, (_, g) = inputs.activations(cfg), inputs.routing(cfg)
        ids = (np.arange(cfg.tokens, dtype=np.int32) % 4)[:, None]
        here = ids < resident
        out = torch.full((cfg.tokens, cfg.hidden), 5.0, dtype=torch.float32, device="cuda")
        pool.reset_page_table()
        pool.materialize(0, np.arange(resident, dtype=np.int32), np.arange(resident, dtype=np.int32))
        args = (0, x.cuda(), torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda(), out)
        pool.expert_ffn(*args, flags=B.FFN_SKIP_UNMAPPED)
        once = out.clone()
        pool.expert_ffn(*args, flags=B.FFN_SKIP_UNMAPPED | B.FFN_ACCUMULATE)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0 and torch.equal(out, once + once)
        some = np.r_[0:64, cfg.tokens - 64:cfg.tokens]
        want = offn.moe_ffn(inputs.bits_u16(x[some].contiguous()), ids[some], np.where(here, g, 0).astype(np.float32)[some],
                            lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
        assert offn.rel_frobenius(once[torch.from_numpy(some).cuda()].cpu().numpy(), want) <= TOL
    finally:
        pool.close()
