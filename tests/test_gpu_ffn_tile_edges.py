"""Edges of the tiled expert FFN's tiles: reductions of one to seven K tiles (shorter than the loads run ahead), a last
column tile of 64, 128 or 192 columns, and the row remainders of every epilogue (ragged, tall by a shared and by an own
block row, shallow), the rows past the segments' end left alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS = [600, 300, 276, 64, 129, 1, 0, 512, 97]


@pytest.mark.parametrize("H,F", [(64, 64), (64, 192), (128, 320), (192, 128), (256, 64), (320, 448), (448, 256)])
def test_tile_edges(H, F):
    import torch
    import paper_2605_05888_amd as hub
    print("tile edges", H, F, flush=True)
    E, M = len(ROWS), sum(ROWS) + 5
    seg = np.concatenate([[0], np.cumsum(ROWS)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(21)
    normal = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    dseg = torch.from_numpy(seg).cuda()
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    y = torch.full((M, H), 7.0, dtype=torch.bfloat16, device="cuda")
    hub.moe_grouped_ffn(xp, dseg, Wg, Wu, Wd, y, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
    for e in range(E):
        x = xp[seg[e]:seg[e + 1]].double()
        want = (torch.nn.functional.silu(x @ Wg[e].double().T) * (x @ Wu[e].double().T)).to(torch.bfloat16).double() @ Wd[e].double().T
        # one rounding of y (2^-9 at most); bf16 steps of `a` that fall on the other side are far rarer than that
        if len(x):
            assert float((y[seg[e]:seg[e + 1]].double() - want).norm() / want.norm()) < 2.0 ** -9, e
    assert bool((y[seg[-1]:] == 7.0).all())
    y2 = torch.full_like(y, 7.0)
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_down(xp, dseg, Wg, Wu, Wd, y2, ws)
    assert torch.equal(y, y2)


# the rows at which an expert changes its geometry, and the rows beside the edges of their blocks
EDGES = [64, 65, 95, 96, 97, 128, 159, 160, 161, 192, 193, 256, 257, 288, 289, 320, 321, 1, 511]


@pytest.mark.parametrize("H,F", [(4096, 192),  # down projection with 256-column tiles
                                 (512, 320),   # with 128-column tiles
                                 (64, 4096), (128, 2048)])
def test_rows_at_the_edges_of_the_geometries(H, F):
    """Against 64-bit arithmetic; and reversed, gathered, added into the tokens' sums and in one launch: the same bits."""
    import torch
    import paper_2605_05888_amd as hub
    print("geometry edges", H, F, flush=True)
    E, M = len(EDGES), sum(EDGES)
    seg = np.concatenate([[0], np.cumsum(EDGES)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(23)
    normal = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    dseg = torch.from_numpy(seg).cuda()
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hub.moe_grouped_ffn(xp, dseg, Wg, Wu, Wd, y, ws)
    for e in range(E):
        x = xp[seg[e]:seg[e + 1]].double()
        want = (torch.nn.functional.silu(x @ Wg[e].double().T) * (x @ Wu[e].double().T)).to(torch.bfloat16).double() @ Wd[e].double().T
        assert float((y[seg[e]:seg[e + 1]].double() - want).norm() / want.norm()) < 2.0 ** -9, EDGES[e]  # (see above)
    rev = torch.cat([torch.arange(lo, hi).flip(0) for lo, hi in zip(seg[:-1], seg[1:])]).cuda()
    y2 = torch.full_like(y, float("nan"))
    hub.moe_grouped_ffn(xp[rev].contiguous(), dseg, Wg, Wu, Wd, y2, ws)
    assert torch.equal(y2, y[rev])
    x = torch.empty_like(xp)
    x[rev] = xp
    y2.fill_(float("nan"))
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_gather(x, 1, dseg, rev.to(torch.int32), Wg, Wu, ws)
    hub.moe_ffn_down(dseg, Wd, y2, ws)
    assert torch.equal(y2, y)
    # added to their tokens' sums (top-1, weight 2: exact doubles); the rows of `a` are still those of xp
    sums, out = torch.empty(M, H, device="cuda"), torch.full_like(y, float("nan"))
    hub.moe_ffn_down_combine(1, dseg, Wd, rev.to(torch.int32), torch.full((M, 1), 2.0, device="cuda"), sums, out, ws)
    assert torch.equal(out[rev], (2.0 * y.float()).to(torch.bfloat16))
    y2.fill_(float("nan"))
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_down(xp, dseg, Wg, Wu, Wd, y2, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
    assert torch.equal(y2, y)
