"""Gathered rows with the shortest reductions whose tiles are chained (the next tile's first loads go out under this one's
last K tile): bit for bit the rows moved first."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [128, 192, 256, 320, 384])
@pytest.mark.parametrize("rows", [40, 100, 200, 290])
def test_short_reductions_gathered(H, rows):
    import torch
    import paper_2605_05888_amd as hub
    print("gather", H, rows, flush=True)
    E, F, K = 48, 4096, 2
    N = E * rows // K
    M = N * K
    g = torch.Generator(device="cuda").manual_seed(31)
    normal = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    x, Wg, Wu, Wd = normal((N, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    seg = torch.arange(E + 1, dtype=torch.int32, device="cuda") * rows
    row = torch.randperm(M, generator=torch.Generator().manual_seed(3)).to(torch.int32).cuda()
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    y, y2 = torch.empty(M, H, dtype=torch.bfloat16, device="cuda"), torch.empty(M, H, dtype=torch.bfloat16, device="cuda")
    hub.moe_grouped_ffn(x[(row // K).long()].contiguous(), seg, Wg, Wu, Wd, y, ws)
    hub.moe_ffn_schedule(hub.BF16, M, H, F, seg, ws)
    hub.moe_ffn_gate_up_gather(x, K, seg, row, Wg, Wu, ws)
    hub.moe_ffn_down(seg, Wd, y2, ws)
    assert torch.equal(y, y2)
