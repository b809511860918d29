"""GPU parity of a second product whose last round of 256 x 256 tiles is split over K: super-tiles of 4 x 8 tiles left over by the 8 XCDs,
from one (eight parts) to five (whole), K of whole steps and not, a buffer without room for the parts, against torch in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2604_02715_amd import binding as B
from paper_2604_02715_amd import harness, inputs
from test_gpu_ffn import TOL

pytestmark = pytest.mark.gpu


def reference(x, w13, w2):
    g, u = x.double() @ w13[0].double(), x.double() @ w13[1].double()
    return (g / (1.0 + torch.exp(-g)) * u).to(torch.bfloat16).double() @ w2.double()


@pytest.mark.parametrize("row_tiles,hidden,ffn,rows_last", [
    (33, 2048, 2112, 1),             # one super-tile left, eight parts; its row tile has a single row
    (38, 2048, 2112, 100),           # two: four parts
    (41, 2048, 2120, 256),           # three: two parts, a partial step
    (48, 2048, 2112, 77),            # four: two parts
    (52, 2048, 2112, 256),           # five: whole
    (34, 2112, 2112, 256),           # two column blocks, the second with one tile of 64 columns: 18 super-tiles
])
def test_last_round(row_tiles, hidden, ffn, rows_last):
    """Two experts, the first with whole row tiles and the second with the rest, a token to one of them."""
    first = 256 * (row_tiles // 2)
    T = 256 * (row_tiles - 1) + rows_last
    cfg = inputs.scaled(inputs.CONFIGS["c1_tiny"], n_experts=2, n_slots=2, top_k=1, tokens=T, hidden=hidden, ffn=ffn)
    pool = harness.ExpertPool(cfg)
    try:
        gen = torch.Generator(device="cuda").manual_seed(row_tiles)
        draw = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
        x = draw(T, hidden).bfloat16()
        w = [((0.02 * draw(2, hidden, ffn)).bfloat16(), (0.02 * draw(ffn, hidden)).bfloat16()) for _ in range(2)]
        for e, (w13, w2) in enumerate(w):
            pool.slot13(e).copy_(w13.view(torch.int16).reshape(-1))
            pool.slot2(e).copy_(w2.view(torch.int16).reshape(-1))
        pool.page_table.copy_(torch.tensor([[0, 1]], dtype=torch.int32))
        who = np.where(np.random.default_rng(row_tiles).permutation(T) < first, 0, 1).astype(np.int32)
        ids, gates = torch.from_numpy(who[:, None]).cuda(), torch.rand(T, 1, generator=gen, device="cuda") + 0.5
        want = torch.empty(T, hidden, dtype=torch.float64, device="cuda")
        for e in range(2):
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
