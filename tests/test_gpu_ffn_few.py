"""GPU parity of calls of up to 64 pairs: the second product with a quarter of K to a wavefront, with and without the first product's
partial sums added up inside it, against the FP64 oracle.  Tolerance as in test_gpu_ffn.py: the sums stay FP32, only their order changes."""
import numpy as np
import pytest
import torch

from oracle import ffn as offn
from paper_2604_02715_amd import inputs
from test_ffn_plan_few import few  # noqa: F401 (fixture)
from test_gpu_ffn import TOL, run_ffn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,path", [
    (dict(tokens=1, top_k=2, hidden=1032, ffn=136), "fused"),                   # a strip of 8 columns, wavefronts of 64, 64, 8 and no k
    (dict(tokens=4, top_k=2, hidden=1024, ffn=512), "fused"),                   # the most tokens and the longest quarters, no tail
    (dict(tokens=3, top_k=3, hidden=2056, ffn=504), "fused"),                   # a tail in the last quarter, eight splits
    (dict(tokens=4, top_k=4, n_experts=16, n_slots=16, hidden=2048, ffn=1016), "fused"),     # quarters of 256 k, the last of them short
    (dict(tokens=1, top_k=8, n_experts=16, n_slots=16, hidden=3080, ffn=776), "fused"),      # of 224 k, a strip of 8 columns
    (dict(tokens=5, top_k=3, hidden=520, ffn=72), "few"),                       # h from the first product
    (dict(tokens=50, top_k=1, hidden=136, ffn=264, routing="zipf"), "few"),     # tiles of 28 rows and of fewer than 16
    (dict(tokens=50, top_k=1, hidden=1000, ffn=520, routing="zipf"), "few"),    # the same in 8 strips, two MFMA tails of 8 k
    (dict(tokens=20, top_k=3, hidden=136, ffn=264), "old"),                     # more than 16 rows are likely where routing is skewed
    (dict(tokens=2, top_k=1, hidden=1024, ffn=2056), "split"),                  # K splits, the last of them short
    (dict(tokens=32, top_k=2, n_experts=64, n_slots=64, hidden=2048, ffn=64), "old"),    # more strips than CUs
])
def test_few_pairs(kw, path, few):
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], **kw)
    p = few.plan(T=cfg.tokens, K=cfg.top_k, E=cfg.n_experts, H=cfg.hidden, F=cfg.ffn, mapped=cfg.n_experts)
    assert path == ("fused" if p.few_fused else "split" if p.few_splits > 1 else "few" if p.few_splits else "old")
    run_ffn_case(cfg, seed=21)


@pytest.mark.parametrize("tokens,top_k", [(4, 8), (4, 3)])
def test_fused_with_more_rows_than_tokens(tokens, top_k):
    """Ids that repeat within a token: 32 and 12 rows of one expert, two passes over its weights and one.  Each listed pair counts, so
    the result is the expert's with the sum of the token's gates."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=tokens, top_k=top_k, hidden=1024, ffn=264)
    pool, dense = build_pool(cfg, seed=22)
    try:
        w13, w2 = dense[0]
        x = inputs.activations(cfg, 0, seed=22)
        g = np.random.default_rng(22).random((tokens, top_k), dtype=np.float32)
        pool.reset_page_table()
        pool.materialize(0, [5], [3])
        out = torch.full((tokens, cfg.hidden), 7.0, device="cuda")
        pool.expert_ffn(0, x.cuda(), torch.full((tokens, top_k), 5, dtype=torch.int32, device="cuda"), torch.from_numpy(g).cuda(), out)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
        want = offn.moe_ffn(inputs.bits_u16(x), np.full((tokens, 1), 5, dtype=np.int32), g.astype(np.float64).sum(axis=1, keepdims=True),
                            lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
        assert offn.rel_frobenius(out.cpu().numpy(), want) <= TOL
    finally:
        pool.close()
