"""Kernel timing spans of the library (benchmark aid): selection of kinds."""
import pytest
import torch

from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import inputs

pytestmark = pytest.mark.gpu


def test_profile_brackets_only_the_selected_kinds():
    from gpu_common import build_pool
    cfg = inputs.CONFIGS["c1_tiny"]
    pool, dense = build_pool(cfg, seed=0)
    try:
        x = inputs.activations(cfg, 0, seed=0).cuda()
        ids, g = inputs.routing(cfg, 0, seed=0)
        idd, gd = torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda()
        out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
        union = inputs.routed_union(ids)
        pool.reset_page_table()

        def step():
            pool.materialize(0, union, list(range(len(union))))
            pool.expert_ffn(0, x, idd, gd, out)

        B.fluxmoe_profile_enable(pool.ctx, True)
        B.fluxmoe_profile_collect(pool.ctx)
        step(); step()
        prof = B.fluxmoe_profile_collect(pool.ctx)
        assert all(prof[k][1] == 2 and prof[k][0] > 0 for k in B.PROFILE_KINDS)

        B.fluxmoe_profile_enable(pool.ctx, True, only_kinds=("decode",))
        step(); step(); step()
        prof = B.fluxmoe_profile_collect(pool.ctx)
        assert prof["decode"][1] == 3 and prof["decode"][0] > 0
        assert all(prof[k] == (0.0, 0) for k in B.PROFILE_KINDS if k != "decode")

        B.fluxmoe_profile_enable(pool.ctx, True, only_kinds=("gemm1_swiglu", "combine"))
        step()
        prof = B.fluxmoe_profile_collect(pool.ctx)
        assert [prof[k][1] for k in B.PROFILE_KINDS] == [0, 0, 1, 0, 1]

        B.fluxmoe_profile_enable(pool.ctx, False)
        step()
        assert all(v == (0.0, 0) for v in B.fluxmoe_profile_collect(pool.ctx).values())
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
    finally:
        pool.close()


def test_a_kind_without_a_kernel_counts_no_launch():
    """Up to 64 pairs the gate/up product's workgroups group the pairs: no launch of kind "grouping" and no time."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=33)
    pool, _ = build_pool(cfg)
    try:
        x = inputs.activations(cfg).cuda()
        ids, g = inputs.routing(cfg)
        idd, gd = torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda()
        out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
        pool.reset_page_table()
        pool.materialize(0, list(range(8)), list(range(8)))
        B.fluxmoe_profile_enable(pool.ctx, True)
        for tokens, launches in ((32, 0), (33, 1)):
            B.fluxmoe_profile_collect(pool.ctx)
            pool.expert_ffn(0, x, idd[:tokens], gd[:tokens], out)
            prof = B.fluxmoe_profile_collect(pool.ctx)
            assert prof["grouping"][1] == launches and (prof["grouping"][0] > 0) == (launches > 0)
            assert all(prof[k][1] == 1 and prof[k][0] > 0 for k in ("gemm1_swiglu", "gemm2", "combine"))
        assert pool.device_errors() == 0
    finally:
        pool.close()


@pytest.mark.parametrize("tokens,hidden,ffn,launches", [
    (64, 256, 128, (0, 1, 1, 0)),              # a few workgroups: no lists, the second product writes the output
    (4100, 512, 512, (1, 1, 1, 0)),            # 128 x 128 tiles: lists
])
def test_kinds_of_the_shared_expert(tokens, hidden, ffn, launches):
    from paper_2604_02715_amd import harness
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=2, shared_expert=True, tokens=tokens, hidden=hidden, ffn=ffn)
    pool = harness.ExpertPool(cfg)
    try:
        s13, s2 = inputs.shared_expert_weights(cfg, 0)
        s13, s2, x = s13.cuda(), s2.cuda(), inputs.activations(cfg).cuda()
        out = torch.zeros((tokens, hidden), dtype=torch.float32, device="cuda")
        B.fluxmoe_profile_enable(pool.ctx, True)
        B.fluxmoe_profile_collect(pool.ctx)
        pool.shared_expert_ffn(s13, s2, x, out)
        prof = B.fluxmoe_profile_collect(pool.ctx)
        kinds = ("grouping", "gemm1_swiglu", "gemm2", "combine")
        assert tuple(prof[k][1] for k in kinds) == launches and all((prof[k][0] > 0) == (prof[k][1] > 0) for k in kinds)
    finally:
        pool.close()
