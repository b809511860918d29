"""GPU parity of the shared expert where gemm_ring_kernel runs it (tiles of 32, 64 and 128 rows, split and unsplit products,
K and N that are multiples of 8 only), against the FP64 oracle.  Tolerance as in test_gpu_ffn.py: the sums are FP32."""
import numpy as np
import pytest
import torch

from oracle import ffn as offn
from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import inputs
from test_gpu_ffn import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,hidden,ffn", [
    (1, 8, 8),              # one partial step, a tile of 8 columns
    (31, 72, 200),          # k tails of 8 in both products
    (32, 1032, 136),        # splits of the first product, the last with a partial step
    (33, 256, 64),          # a second row tile of one row; the second product is a single step
    (64, 2048, 512),        # splits, whole steps
    (211, 2048, 520),       # rows that leave wavefronts without any
    (257, 520, 1032),       # both products with tails
    (130, 3000, 1000),      # tiles of 64 rows
    (600, 1024, 1536),      # tiles of 128 rows
    (241, 1504, 2776),      # second product split
])
def test_shared_expert_in_the_ring_kernel(tokens, hidden, ffn):
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=2, shared_expert=True, tokens=tokens, hidden=hidden, ffn=ffn)
    pool, _ = build_pool(cfg)
    try:
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


def test_infinite_weights_in_the_last_rows_stay_where_they_belong():
    """The pieces past the end of K are zeros, not a repeated row: an infinite weight in the last k row of either product makes
    the columns infinite (or not a number) that it makes so in 64 bits, and no others."""
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
