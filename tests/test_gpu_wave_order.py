"""Waves of one layer through two slot halves without a release between load and load: the second wave's materialize
follows the first wave's FFN on another stream at once.  The FFN, held back on its stream, must still see the first wave
only (its experts would otherwise be taken twice, or read before they are decoded), and a third load into the first half
must wait for the FFN that read it and not overtake it."""
import numpy as np
import pytest
import torch

from oracle import ffn as offn
from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import inputs

pytestmark = pytest.mark.gpu


def test_next_wave_is_loaded_while_the_last_one_waits_to_run():
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=12, n_slots=8, tokens=48, top_k=4)
    pool, dense = build_pool(cfg)
    try:
        w13, w2 = dense[0]
        x = inputs.activations(cfg)
        ids, g = inputs.routing(cfg)
        xd, idd, gd = x.cuda(), torch.from_numpy(ids).cuda(), torch.from_numpy(g).cuda()
        want = offn.moe_ffn(inputs.bits_u16(x), ids, g, lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
        waves = [(np.arange(4 * i, 4 * i + 4), 4 * (i & 1) + np.arange(4)) for i in range(3)]
        results = []
        for load, infer, delay in ((None, None, 0), (torch.cuda.Stream(), torch.cuda.Stream(), 300000),
                                   (torch.cuda.Stream(), torch.cuda.Stream(), 0)):
            infer = infer or torch.cuda.current_stream()
            out = torch.full((cfg.tokens, cfg.hidden), float("nan"), device="cuda")
            pool.poison_slots()
            pool.reset_page_table()
            torch.cuda.synchronize()
            for i, (e, s) in enumerate(waves):
                pool.materialize(0, e, s, load)
                if i:
                    pool.release(0, waves[i - 1][0], infer)
                if delay:
                    with torch.cuda.stream(infer):
                        torch.cuda._sleep(delay)
                pool.expert_ffn(0, xd, idd, gd, out, B.FFN_SKIP_UNMAPPED | (B.FFN_ACCUMULATE if i else 0), infer)
            pool.release(0, waves[-1][0], infer)
            torch.cuda.synchronize()
            assert pool.device_errors() == 0
            assert (pool.page_table == -1).all()
            assert offn.rel_frobenius(out.cpu().numpy(), want) <= 1e-3
            results.append(out.cpu().numpy())
        assert all(np.array_equal(r, results[0]) for r in results)
    finally:
        pool.close()
