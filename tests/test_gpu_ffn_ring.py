"""GPU parity of the shared expert where gemm_ring_kernel runs it (tiles of 32, 64 and 128 rows, split and unsplit products,
K and N that are multiples of 8 only) and past it, against the FP64 oracle.  Tolerance as in test_gpu_ffn.py: the sums are FP32."""
import numpy as np
import pytest
import torch

from oracle import ffn as offn
from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import inputs
from test_ffn_plan_shared import rules  # noqa: F401 (fixture)
from test_gpu_ffn import TOL

pytestmark = pytest.mark.gpu


def scratch_of(pool):
    return pool.ws_bytes - int(pool.sizes.pool_workspace_bytes)


def check_shared(rules, tokens, hidden, ffn, plan):
    """One call that overwrites and one that accumulates against the oracle; the plan is (rows of a tile and splits of the first
    product, of the second) of gemm_ring_kernel, or (0, m_tile, tiled, splits of the second)."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=2, shared_expert=True, tokens=tokens, hidden=hidden, ffn=ffn)
    pool, _ = build_pool(cfg)
    try:
        p = rules.shared(tokens, hidden, ffn, scratch_of(pool))
        assert ((p.ring1, p.ksplit1, p.ring2, p.ksplit) if p.ring1 else (0, p.m_tile, p.tiled, p.ksplit)) == plan
        s13, s2 = inputs.shared_expert_weights(cfg, 0)
        x = inputs.activations(cfg)
        s13d, s2d, xd = s13.cuda(), s2.cuda(), x.cuda()
        guard = torch.full((tokens + 2, hidden), 5.0, dtype=torch.float32, device="cuda")
        out = guard[1:tokens + 1]
        pool.shared_expert_ffn(s13d, s2d, xd, out)
        once = out.clone()
        pool.shared_expert_ffn(s13d, s2d, xd, out, B.FFN_ACCUMULATE)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
        want = offn.moe_ffn(inputs.bits_u16(x), np.zeros((tokens, 1), dtype=np.int32), np.ones((tokens, 1), dtype=np.float32),
                            lambda e: (inputs.bits_u16(s13), inputs.bits_u16(s2)))
        assert offn.rel_frobenius(once.cpu().numpy(), want) <= TOL
        assert torch.equal(out, once + once)
        assert bool((guard[0] == 5.0).all()) and bool((guard[-1] == 5.0).all())      # nothing past the rows
    finally:
        pool.close()


@pytest.mark.parametrize("tokens,hidden,ffn,plan", [
    (1, 8, 8, (32, 1, 32, 1)),                  # one partial step, a tile of 8 columns
    (31, 72, 200, (32, 1, 32, 1)),              # k tails of 8 in both products
    (32, 1032, 136, (32, 6, 32, 1)),            # splits of the first product, the last with a partial step
    (33, 256, 64, (32, 1, 32, 1)),              # a second row tile of one row; the second product is a single step
    (64, 2048, 512, (32, 8, 32, 1)),            # splits, whole steps
    (211, 2048, 520, (64, 7, 32, 1)),           # rows that leave wavefronts without any
    (257, 520, 1032, (32, 1, 64, 6)),           # both products with tails
    (130, 3000, 1000, (128, 8, 32, 1)),
    (600, 1024, 1536, (64, 1, 32, 1)),
    (241, 1504, 2776, (64, 1, 64, 5)),          # second product split
    (129, 1824, 1440, (128, 5, 128, 8)),        # tiles of 128 rows in both, split, tails
    (1359, 136, 1128, (128, 1, 128, 6)),        # the first whole
    (9000, 256, 192, (128, 1, 128, 1)),         # both whole: the second writes the output
    (8487, 168, 72, (128, 1, 128, 1)),          # and with tails
    (9116, 48, 16, (64, 1, 64, 1)),             # less than a step of either
])
def test_shared_expert_in_the_ring_kernel(rules, tokens, hidden, ffn, plan):
    check_shared(rules, tokens, hidden, ffn, plan)


@pytest.mark.parametrize("tokens,hidden,ffn,plan", [
    (4100, 512, 512, (0, 128, 1, 1)),           # tiles of 128 x 128, a last row tile of four rows
    (9000, 520, 520, (0, 256, 1, 1)),           # of 256 x 256 with partial steps
])
def test_shared_expert_past_the_ring_kernel(rules, tokens, hidden, ffn, plan):
    """Lists of every token in order, and the LDS-direct second product writes the output itself."""
    check_shared(rules, tokens, hidden, ffn, plan)


def test_what_lies_behind_the_operands_stays_out():
    """The pieces past the end of K are zeros: rows behind the weights and behind a token's row are infinite here.  A token's own
    infinities make its row infinite or not a number, and no other."""
    from gpu_common import build_pool
    tokens, hidden, ffn = 129, 1824, 1448
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=2, shared_expert=True, tokens=tokens, hidden=hidden, ffn=ffn)
    pool, _ = build_pool(cfg)
    try:
        s13, s2 = inputs.shared_expert_weights(cfg, 0)
        x = inputs.activations(cfg).clone()
        x[100] = float("inf")
        behind = lambda t, cols: torch.cat([t.reshape(-1), torch.full((64 * cols,), float("inf"), dtype=t.dtype)]).cuda()
        out = torch.zeros((tokens, hidden), dtype=torch.float32, device="cuda")
        pool.shared_expert_ffn(behind(s13, ffn), behind(s2, hidden), x.cuda(), out)
        torch.cuda.synchronize()
        others = [t for t in range(tokens) if t != 100]
        assert not bool(torch.isfinite(out[100]).any())
        want = offn.moe_ffn(inputs.bits_u16(x[others].contiguous()), np.zeros((tokens - 1, 1), dtype=np.int32), np.ones((tokens - 1, 1), dtype=np.float32),
                            lambda e: (inputs.bits_u16(s13), inputs.bits_u16(s2)))
        assert offn.rel_frobenius(out[others].cpu().numpy(), want) <= TOL
    finally:
        pool.close()


def test_infinite_weights_in_the_last_rows_stay_where_they_belong():
    """The pieces past the end of K are zeros, not a repeated row: an infinite weight in the last k row of the second product makes
    its own column infinite (or not a number), and no other."""
    from gpu_common import build_pool
    tokens, hidden, ffn = 40, 72, 200
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=2, shared_expert=True, tokens=tokens, hidden=hidden, ffn=ffn)
    pool, _ = build_pool(cfg)
    try:
        s13, s2 = inputs.shared_expert_weights(cfg, 0)
        s13, s2 = s13.clone(), s2.clone()
        s2.view(ffn, hidden)[ffn - 1, 5] = float("inf")
        x = inputs.activations(cfg)
        out = torch.zeros((tokens, hidden), dtype=torch.float32, device="cuda")
        pool.shared_expert_ffn(s13.cuda(), s2.cuda(), x.cuda(), out)
        torch.cuda.synchronize()
        bad = ~torch.isfinite(out.cpu())
        assert bool(bad[:, 5].all()) and int(bad.sum()) == tokens
    finally:
        pool.close()
