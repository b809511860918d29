"""Waves on several streams under stream capture: the recorded graph must hold the order that the calls have outside
capture, above all that a wave's FFN reads the page table before the next wave's entries appear there.  The inference
stream is held back before every FFN inside the graph, so that a load without that edge would overtake it and its experts
be taken twice.  Every replay is compared with an eager pass of another context, with eager work in between."""
import numpy as np
import pytest
import torch

from oracle import ffn as offn
from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import harness, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens", [16, 48, 3600])          # grouped by the first product, by one workgroup, by several
def test_a_captured_pass_in_waves_replays_as_the_eager_one(tokens):
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=12, n_slots=8, n_layers=2, tokens=tokens, top_k=4, ffn=128)
    routings = [inputs.routing(cfg, layer) for layer in range(2)]
    xs = [inputs.activations(cfg, layer) for layer in range(2)]
    pools, proxies = [], []
    try:
        for _ in range(2):                                   # one pass is eager, the other pool's first pass is captured
            pool, dense = build_pool(cfg)
            pools.append(pool)
            pool.reset_page_table()
            pool.poison_slots()
            outs = [torch.full((tokens, cfg.hidden), float("nan"), device="cuda") for _ in range(2)]
            proxies.append(harness.StreamingProxy(pool, routings, [x.cuda() for x in xs], outs))
        eager, captured = proxies
        assert [len(waves) for _, waves in captured.plan] == [3, 3]
        torch.cuda.synchronize()
        eager.run_pass()
        torch.cuda.synchronize()
        for layer in range(2):
            w13, w2 = dense[layer]
            some = slice(0, min(tokens, 48))
            want = offn.moe_ffn(inputs.bits_u16(xs[layer][some]), routings[layer][0][some], routings[layer][1][some],
                                lambda e: (inputs.bits_u16(w13[e]), inputs.bits_u16(w2[e])))
            assert offn.rel_frobenius(eager.outs[layer][some].cpu().numpy(), want) <= 1e-3

        graph = torch.cuda.CUDAGraph()
        infer, load = captured.infer_stream, captured.load_stream
        with torch.cuda.graph(graph, stream=infer, capture_error_mode="relaxed"):
            load.wait_stream(infer)
            captured.run_pass(ffn_delay_cycles=300000)
            infer.wait_stream(load)
        for _ in range(4):
            for out in captured.outs:
                out.fill_(float("nan"))
            pools[1].poison_slots()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(captured.outs, eager.outs))
            assert (pools[1].page_table == -1).all()
        assert pools[0].device_errors() == 0 and pools[1].device_errors() == 0
    finally:
        for pool in pools:
            pool.close()


def test_a_captured_load_leaves_the_staging_half_guarded():
    """A load that reads the staging half is still waiting to run when another load of its layer, without host-tier blocks,
    is captured; the next fetch into that half must wait for the first one all the same."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_layers=3, host_fraction=0.15)     # the down tensors of experts 0 to 3
    pool, dense = build_pool(cfg, host_fraction=cfg.host_fraction)
    try:
        pool.bind_staging(64 << 20)
        pool.reset_page_table()
        pool.poison_slots()
        load, side, copy = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        pool.prefetch_host(0, [0, 1, 2, 3], copy)
        torch.cuda.synchronize()
        with torch.cuda.stream(load):
            torch.cuda._sleep(400000000)
        pool.materialize(0, [0, 1, 2, 3], [0, 1, 2, 3], load)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            graph.capture_begin(capture_error_mode="relaxed")
            pool.materialize(0, [6, 7], [6, 7], side)
            graph.capture_end()
        pool.prefetch_host(2, [0, 1, 2, 3], copy)
        assert not load.query()                              # or the wait was not needed
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
        for e in (0, 1, 2, 3, 6, 7):
            assert torch.equal(pool.slot13(e).cpu(), dense[0][0][e].reshape(-1).view(torch.int16))
            assert torch.equal(pool.slot2(e).cpu(), dense[0][1][e].reshape(-1).view(torch.int16))
        pool.materialize(2, [0, 1, 2, 3], [3, 2, 1, 0], load)
        torch.cuda.synchronize()
        assert pool.device_errors() == 0
        for e in range(4):
            assert torch.equal(pool.slot2(3 - e).cpu(), dense[2][1][e].reshape(-1).view(torch.int16))
    finally:
        pool.close()


def test_slots_last_read_before_a_capture_are_loaded_inside_it():
    """The slots that an eager, timed FFN call read are taken by a captured load of another layer, after the layer's experts
    were loaded elsewhere and its FFN captured: the load waits for the captured call, and not for the eager one, whose event
    was recorded on the same stream and is refused inside a capture."""
    from gpu_common import build_pool
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_layers=2, n_slots=16)
    pool, _ = build_pool(cfg)
    try:
        pool.reset_page_table()
        xs = [inputs.activations(cfg, layer).cuda() for layer in range(2)]
        routings = [[torch.from_numpy(r).cuda() for r in inputs.routing(cfg, layer)] for layer in range(2)]
        outs = [torch.zeros((cfg.tokens, cfg.hidden), device="cuda") for _ in range(2)]
        every = np.arange(8)
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        pool.materialize(0, every, every)
        B.fluxmoe_profile_enable(pool.ctx, True)
        pool.expert_ffn(0, xs[0], *routings[0], outs[0], stream=side)
        B.fluxmoe_profile_enable(pool.ctx, False)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
            pool.materialize(0, every, 8 + every, side)
            pool.expert_ffn(0, xs[0], *routings[0], outs[0], stream=side)
            pool.materialize(1, every, every, side)
            pool.expert_ffn(1, xs[1], *routings[1], outs[1], stream=side)
        results = []
        for _ in range(3):
            pool.poison_slots()
            for out in outs:
                out.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            results.append([out.clone() for out in outs])
        pool.expert_ffn(0, xs[0], *routings[0], outs[0])         # all sixteen experts are resident now
        pool.expert_ffn(1, xs[1], *routings[1], outs[1])
        torch.cuda.synchronize()
        assert all(torch.equal(got, out) for result in results for got, out in zip(result, outs))
        assert pool.device_errors() == 0
    finally:
        pool.close()
