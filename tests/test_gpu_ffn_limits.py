"""The expert FFN at the sizes where 32-bit offsets end."""
import numpy as np
import pytest
import torch

from oracle import ffn as offn
from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import harness, inputs
from test_gpu_ffn import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant,top_k,ffn", [
    ("2", 17, 2048),        # LDS-direct kernels, the second product's workgroups walk
    ("2", 5, 8192),         # one tile each
    ("1", 5, 8192),         # four wavefronts
    ("4", 9, 8192),         # register-staged loads, four wavefronts: offsets counted in elements
])
def test_rows_of_h_past_four_gigabytes(variant, top_k, ffn, monkeypatch):
    """Every token on every expert: the last expert's rows of the SwiGLU product lie past 2^32 bytes (elements for the last
    variant) from the buffer's start.  Some tokens against the oracle."""
    from gpu_common import build_pool
    monkeypatch.setenv("FLUXMOE_FFN_TILED_WAVES", variant)
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], tokens=65535, top_k=top_k, n_experts=top_k, n_slots=top_k, hidden=64, ffn=ffn)
    pool, dense = build_pool(cfg)
    try:
        w13, w2 = dense[0]
        x = inputs.activations(cfg)
        ids, g = inputs.routing(cfg)
        out = torch.zeros((cfg.tokens, cfg.hidden), dtype=torch.float32, device="cuda")
        pool.reset_page_table()
        pool.materialize(0, np.arange(top_k), np.arange(top_k))
        pool.expert_ffn(0, x.cuda(), torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda(), out)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
        some = np.linspace(0, cfg.tokens - 1, 40).astype(int)
        want = offn.moe_ffn(inputs.bits_u16(x[torch.from_numpy(some)]), ids[some], g[some],
                            lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
        assert offn.rel_frobenius(out.cpu().numpy()[some], want) <= TOL
    finally:
        pool.close()


def test_tokens_past_four_gigabytes_are_refused():
    """T * hidden * 2 bytes: the limit of the routed call holds for the shared expert too; nothing is enqueued."""
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=1, hidden=32832, ffn=64, tokens=1, top_k=1, shared_expert=True)
    pool = harness.ExpertPool(cfg)
    try:
        some = pool.slots13.data_ptr()
        tokens = (1 << 32) // (2 * cfg.hidden) + 1
        for call in (lambda: B.fluxmoe_shared_expert_ffn(pool.ctx, some, some, some, tokens, some, 0, 0),
                     lambda: B.fluxmoe_expert_ffn(pool.ctx, 0, some, tokens, some, some, 1, some, some, 0, 0)):
            with pytest.raises(B.FluxmoeError) as ei:
                call()
            assert ei.value.status == -1 and "4 GiB" in str(ei.value)
    finally:
        pool.close()
