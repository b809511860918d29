"""GPU parity of a second product whose last round of 256 x 256 tiles is split over K: super-tiles of 4 x 8 tiles left over by the 8 XCDs,
from one (eight parts) to five (whole), K of whole steps and not, a buffer without room for the parts, against torch in 64 bits."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import harness, inputs
from test_gpu_ffn import TOL

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")


def reference(x, w13, w2):
    g, u = x.double() @ w13[0].double(), x.double() @ w13[1].double()
    return (g / (1.0 + torch.exp(-g)) * u).to(torch.bfloat16).double() @ w2.double()


CASES = [
    (2, 33, 2048, 3136, 1),          # one super-tile left, eight parts; its row tile has a single row
    (2, 38, 2048, 3136, 100),        # two: four parts
    (2, 41, 2048, 3272, 256),        # three: two parts, a partial step
    (2, 48, 2048, 3136, 77),         # four: two parts
    (2, 52, 2048, 3136, 256),        # five: whole
    (2, 34, 2112, 3136, 256),        # two column blocks, the second with one tile of 64 columns: 18 super-tiles
    (41, 41, 2048, 3136, 30),        # a row tile an expert and 1.6 GB of weights: they pass the caches by
]


@pytest.mark.parametrize("experts,row_tiles,hidden,ffn,rows_last", CASES)
def test_the_plan_splits_the_last_round(experts, row_tiles, hidden, ffn, rows_last, tmp_path):
    T = 256 * (row_tiles - 1) + rows_last
    (tmp_path / "m.cpp").write_text("""
#include "ffn_plan.h"
int main() {
    const fluxmoe::FfnShape c{%d, %d, %d, 256, 2, true};
    const fluxmoe::FfnPlan p = fluxmoe::plan_ffn(c, %d, 1, fluxmoe::ffn_bytes(c, %d, 1), %d);
    const bool pays = fluxmoe::last_round_pays(%d, c.E, c.E, c.H, c.F);
    return p.tail && pays == %d && p.m_tile == 256 && fluxmoe::weights_stream(c.E, c.H, c.F, %d, 256) == (c.E > 2) ? 0 : 1;
}
""" % (experts, hidden, ffn, T, T, experts, T, row_tiles != 52, T))
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    subprocess.run([str(tmp_path / "m")], check=True)


def test_both_sides_of_the_lines(tmp_path):
    (tmp_path / "m.cpp").write_text("""
#include "ffn_plan.h"
using namespace fluxmoe;
int main() {
    const FfnShape at{2, 2048, 3072, 256, 2, true}, below{2, 2048, 3064, 256, 2, true};
    if (!plan_ffn(at, 9000, 1).tail || plan_ffn(below, 9000, 1).tail) return 1;
    // one expert: the number of row tiles is known
    for (uint64_t n = 1; n <= 200; ++n) {
        const uint64_t rest = (n + 3) / 4 % 8;
        if (last_round_pays(256 * n - 255, 0, 1, 2048, 3072) != (rest >= 1 && rest <= 4)) return 2;
        if (last_round_pays(256 * n, 1, 1, 4096, 3072) != (rest % 4 == 1 || rest % 4 == 2)) return 3;
    }
    // 8 of H 4096, 936 rows each: 32 row tiles, a whole round; short K does not wager on other routings, long K does
    if (last_round_pays(7488, 8, 8, 4096, 3584) || !last_round_pays(7488, 8, 8, 4096, 14336)) return 4;
    if (!last_round_pays(8192, 0, 8, 4096, 14336) || last_round_pays(0, 0, 8, 4096, 14336) || last_round_pays(1, 1, 8, 4096, 14336)) return 5;
    return 0;
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    assert subprocess.run([str(tmp_path / "m")]).returncode == 0


@pytest.mark.gpu
@pytest.mark.parametrize("experts,row_tiles,hidden,ffn,rows_last", CASES)
def test_last_round(experts, row_tiles, hidden, ffn, rows_last):
    """The experts with whole row tiles but for the last, which has the rest; a token to one of them."""
    each = 256 * (row_tiles // experts)
    T = 256 * (row_tiles - 1) + rows_last
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=experts, n_slots=experts, top_k=1, tokens=T, hidden=hidden, ffn=ffn)
    pool = harness.ExpertPool(cfg)
    try:
        gen = torch.Generator(device="cuda").manual_seed(row_tiles)
        draw = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
        x = draw(T, hidden).bfloat16()
        w = [((0.02 * draw(2, hidden, ffn)).bfloat16(), (0.02 * draw(ffn, hidden)).bfloat16()) for _ in range(experts)]
        for e, (w13, w2) in enumerate(w):
            pool.slot13(e).copy_(w13.view(torch.int16).reshape(-1))
            pool.slot2(e).copy_(w2.view(torch.int16).reshape(-1))
        pool.page_table.copy_(torch.arange(experts, dtype=torch.int32)[None])
        who = np.minimum(np.random.default_rng(row_tiles).permutation(T) // each, experts - 1).astype(np.int32)
        ids, gates = torch.from_numpy(who[:, None]).cuda(), torch.rand(T, 1, generator=gen, device="cuda") + 0.5
        want = torch.empty(T, hidden, dtype=torch.float64, device="cuda")
        for e in range(experts):
            t = torch.from_numpy(np.flatnonzero(who == e)).cuda()
            want[t] = gates[t].double() * reference(x[t], *w[e])
        room = pool.ws_bytes - int(pool.sizes.pool_workspace_bytes)
        outs = []
        for scratch in (room, T * (ffn * 2 + hidden * 4) + (1 << 20)):       # the second: sums of one product and no more
            assert scratch <= room
            B.fluxmoe_bind_arenas(pool.ctx, pool.slots13.data_ptr(), pool.slots2.data_ptr(), pool.workspace.data_ptr(),
                                  int(pool.sizes.pool_workspace_bytes) + scratch)
            pool.workspace[int(pool.sizes.pool_workspace_bytes):].fill_(0x7F)
            out = torch.full((T, hidden), 7.0, device="cuda")
            pool.expert_ffn(0, x, ids, gates, out)
            torch.cuda.synchronize()
            assert pool.device_errors() == 0
            assert (pool.workspace[int(pool.sizes.pool_workspace_bytes) + scratch:] == 0x7F).all()
            assert float((out.double() - want).norm() / want.norm()) <= TOL
            # no row is worse than the others: a tile with a missing or doubled part would be
            assert float(((out.double() - want).norm(dim=1) / want.norm(dim=1)).max()) <= 10 * TOL
            outs.append(out)
        assert torch.equal(outs[0], outs[1]) == (row_tiles == 52)            # parts end a sum elsewhere
    finally:
        pool.close()


@pytest.mark.gpu
@pytest.mark.parametrize("experts,row_tiles,rows_last,top_k", [
    (2, 38, 100, 1),                 # a token's rows change between whole tiles and those in four parts within the second expert
    (2, 66, 100, 1),                 # 16740 pairs: grouped in chunks
    (5, 42, 100, 2),                 # several experts' last tiles in the last round, two rows a token
])
def test_the_same_bits_on_every_call(experts, row_tiles, rows_last, top_k):
    hidden, ffn = 2048, 3136
    T = (256 * (row_tiles - 1) + rows_last) // top_k
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=experts, n_slots=experts, top_k=top_k, tokens=T, hidden=hidden, ffn=ffn)
    pool = harness.ExpertPool(cfg)
    try:
        gen = torch.Generator(device="cuda").manual_seed(row_tiles)
        draw = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
        x = draw(T, hidden).bfloat16()
        w = [((0.02 * draw(2, hidden, ffn)).bfloat16(), (0.02 * draw(ffn, hidden)).bfloat16()) for _ in range(experts)]
        for e, (w13, w2) in enumerate(w):
            pool.slot13(e).copy_(w13.view(torch.int16).reshape(-1))
            pool.slot2(e).copy_(w2.view(torch.int16).reshape(-1))
        pool.page_table.copy_(torch.arange(experts, dtype=torch.int32)[None])
        ids = draw(T, experts).topk(top_k).indices.int().contiguous()
        gates = torch.rand(T, top_k, generator=gen, device="cuda") + 0.5
        want = torch.zeros(T, hidden, dtype=torch.float64, device="cuda")
        for e in range(experts):
            t, k = (ids == e).nonzero(as_tuple=True)
            want[t] += gates[t, k, None].double() * reference(x[t], *w[e])
        first = None
        for call in range(8):
            out = torch.full((T, hidden), 7.0, device="cuda")
            pool.expert_ffn(0, x, ids, gates, out)
            torch.cuda.synchronize()
            if first is None:
                first = out
                assert pool.device_errors() == 0
                assert float(((out.double() - want).norm(dim=1) / want.norm(dim=1)).max()) <= 10 * TOL
            assert torch.equal(out, first), f"call {call}"
    finally:
        pool.close()
