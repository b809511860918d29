"""The standalone-decompression setting of Sec. 6.3 Exp#3 (Tab. "standalone_decompression"): one GPU's
rank-local shard of one layer - Mixtral-8x7B 8 / 2 = 4 experts, Qwen3-Next 512 / 4 = 128, GLM-4.5 160 / 8 = 20 -
materialized whole (routing-independent), the two tensor types on two streams as the paper's loading path
issues them (Sec. 5).  Every slot byte must equal the original tensor, the page table the placement model,
blocks sampled from the pool what the oracle decodes from the same bytes; and the two-stream call must leave
exactly what the one-stream call leaves."""
import numpy as np
import pytest
import torch

from oracle import codec, paging
from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import harness, inputs

pytestmark = pytest.mark.gpu

SHARDS = {"c2_mixtral": 4, "c3_qwen3next": 128, "c4_glm45": 20}


@pytest.mark.parametrize("name", sorted(SHARDS))
def test_rank_local_shard_two_streams(name):
    n_exp = SHARDS[name]
    cfg = inputs.scaled(inputs.CONFIGS[name], n_experts=n_exp, n_slots=n_exp, shared_expert=False)
    pool = harness.ExpertPool(cfg)
    try:
        w13, w2 = harness.make_layer_on_host(cfg, 0, 0, gen_device="cuda")
        blob = pool.encode_layer(0, w13, w2)
        pool.bind_layer(0, blob)
        ids = np.arange(n_exp, dtype=np.int32)
        slots = inputs.slot_permutation(n_exp, name, "exp3-test")
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        model = paging.PagedSlots(1, n_exp, n_exp, cfg.hidden, cfg.ffn, track_bytes=False)
        model.materialize(0, ids, slots, None, None)
        results = []
        for two in (True, False, True):
            pool.poison_slots(0x7FC1)
            pool.reset_page_table()
            torch.cuda.synchronize()
            if two:
                pool.materialize_two_streams(0, ids, slots, s1, s2)
            else:
                pool.materialize(0, ids, slots, s1)
            # the layer's load event is what a consumer waits for: the FFN path does so inside the library;
            # here the device is synchronised
            torch.cuda.synchronize()
            assert pool.device_errors() == 0
            assert np.array_equal(pool.page_table.cpu().numpy(), model.page_table)
            for e, s_ in zip(ids, slots):
                assert torch.equal(pool.slot13(int(s_)), w13[int(e)].reshape(-1).view(torch.int16).cuda()), \
                    "%s expert %d: type-1 slot differs (two streams: %s)" % (name, e, two)
                assert torch.equal(pool.slot2(int(s_)), w2[int(e)].reshape(-1).view(torch.int16).cuda()), \
                    "%s expert %d: type-2 slot differs (two streams: %s)" % (name, e, two)
            results.append(two)
        # sampled blocks of both types against the oracle's decoding of the same pool bytes
        blocks = blob.numpy().reshape(-1, 4096)
        rng = np.random.default_rng(3)
        for d in (1, 2, 1, 2):
            e = int(rng.integers(n_exp))
            b0, nb = B.fluxmoe_tensor_blocks(pool.ctx, 0, d, e)
            k = int(rng.integers(nb))
            e0, n, parts = codec.decode_blocks(blocks[b0 + k:b0 + k + 1], B.fluxmoe_code_lengths(pool.ctx, 0, d))
            view = pool.slot13(int(slots[e])) if d == 1 else pool.slot2(int(slots[e]))
            got = view[int(e0[0]):int(e0[0]) + int(n[0])].cpu().numpy().view(np.uint16)
            assert np.array_equal(got, parts[0])
    finally:
        pool.close()


@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("n_exp", [8, 160])       # a command inside the kernel arguments, and one that is uploaded
def test_two_streams_behind_copies(n_exp, staged):
    """Host-tier blocks and the job list reach the second stream's decode through the fork from the first: blocks copied
    by the call itself on the first stream, or on a copy stream that only the first stream waits for.  Other experts with
    each call, so that what a buffer held before would be the wrong bytes."""
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=n_exp, n_slots=n_exp // 2, host_fraction=0.75)
    pool = harness.ExpertPool(cfg)
    try:
        w13, w2 = harness.make_layer_on_host(cfg)
        _, n_host = pool.bind_layer(0, pool.encode_layer(0, w13, w2), cfg.host_fraction)
        pool.bind_staging(2 * (n_host + 1) * 4096)
        s1, s2, copy = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        pool.reset_page_table()
        for call in range(6):
            ids = np.sort(np.random.default_rng(call).permutation(n_exp)[:n_exp // 2]).astype(np.int32)
            slots = inputs.slot_permutation(n_exp // 2, "behind copies", call)
            pool.poison_slots()
            torch.cuda.synchronize()
            if staged:
                pool.prefetch_host(0, ids, copy)
            pool.materialize_two_streams(0, ids, slots, s1, s2)
            torch.cuda.synchronize()
            assert pool.device_errors() == 0
            for e, s_ in zip(ids, slots):
                assert torch.equal(pool.slot13(int(s_)).cpu(), w13[int(e)].reshape(-1).view(torch.int16))
                assert torch.equal(pool.slot2(int(s_)).cpu(), w2[int(e)].reshape(-1).view(torch.int16))
    finally:
        pool.close()
