"""Down projection into rows so wide that those of one tile take more than 4 GiB, more than the byte count that bounds its stores
can hold."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,H", [(330, 64 * 105469),    # a full row tile and one of 74 rows; 318 rows fit into 4 GiB
                                 (320, 64 * 105469),    # a tall tile with two block rows more
                                 (288, 64 * 116600),    # one block row more
                                 (300, 64 * 131073),    # 256 rows do not fit
                                 (40, 2 ** 26 - 64),    # 32 rows fit, of all that go through tiles the widest
                                 (40, 2 ** 26),         # 32 rows do not fit
                                 (330, 2 ** 26)])
def test_down(M, H):
    import torch
    import paper_2605_05888_amd as hub
    F = 64
    assert M * H * 2 > 2 ** 32
    print("wide rows", M, H, F, flush=True)
    g = torch.Generator(device="cuda").manual_seed(51)
    Wd = torch.empty((1, H, F), dtype=torch.bfloat16, device="cuda").normal_(0.0, F ** -0.5, generator=g)
    seg = torch.tensor([0, M], dtype=torch.int32, device="cuda")
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=1, F=F), dtype=torch.uint8, device="cuda")
    a = ws[:M * F * 2].view(torch.bfloat16).view(M, F)   # the activation lies at the workspace's start
    a.normal_(0.0, 1.0, generator=g)
    y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hub.moe_ffn_schedule(hub.BF16, M, H, F, seg, ws)
    hub.moe_ffn_down(seg, Wd, y, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, 1, ws)
    step = 1 << 19
    for c in range(0, H, step):
        want = a.float() @ Wd[0, c:c + step].float().T
        assert float((y[:, c:c + step].float() - want).norm() / want.norm()) < 2.0 ** -9, c   # (one rounding of y)


def test_down_into_sums():
    import torch
    import paper_2605_05888_amd as hub
    N, H, F = 40, 2 ** 26, 64
    print("wide rows, sums", flush=True)
    g = torch.Generator(device="cuda").manual_seed(52)
    Wd = torch.empty((1, H, F), dtype=torch.bfloat16, device="cuda").normal_(0.0, F ** -0.5, generator=g)
    seg = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=N, H=H, E=1, F=F), dtype=torch.uint8, device="cuda")
    a = ws[:N * F * 2].view(torch.bfloat16).view(N, F)
    a.normal_(0.0, 1.0, generator=g)
    y, out = torch.empty((N, H), dtype=torch.bfloat16, device="cuda"), torch.full((N, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hub.moe_ffn_schedule(hub.BF16, N, H, F, seg, ws)
    hub.moe_ffn_down(seg, Wd, y, ws)
    rev = torch.arange(N - 1, -1, -1, device="cuda")
    # top-1, weight 2: exact doubles
    hub.moe_ffn_down_combine(1, seg, Wd, rev.to(torch.int32), torch.full((N, 1), 2.0, device="cuda"), torch.empty((N, H), device="cuda"), out, ws)
    for m in range(N):
        assert torch.equal(out[N - 1 - m], 2 * y[m]), m


@pytest.mark.parametrize("M", [40, 257])
@pytest.mark.parametrize("gather", [False, True])
def test_gate_up(M, gather):
    import torch
    import paper_2605_05888_amd as hub
    H, F = 64, 2 ** 26
    print("wide rows, gate/up", M, gather, flush=True)
    g = torch.Generator(device="cuda").manual_seed(53)
    normal = lambda shape, std: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, Wg, Wu = normal((M, H), 1.0), normal((1, F, H), H ** -0.5), normal((1, F, H), H ** -0.5)
    seg = torch.tensor([0, M], dtype=torch.int32, device="cuda")
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=1, F=F), dtype=torch.uint8, device="cuda")
    a = ws[:M * F * 2].view(torch.bfloat16).view(M, F)
    a.fill_(float("nan"))
    hub.moe_ffn_schedule(hub.BF16, M, H, F, seg, ws)
    if gather:
        hub.moe_ffn_gate_up_gather(x, 1, seg, torch.arange(M, dtype=torch.int32, device="cuda"), Wg, Wu, ws)
    else:
        hub.moe_ffn_gate_up(x, seg, Wg, Wu, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, 1, ws)
    step = 1 << 19
    for c in range(0, F, step):
        want = torch.nn.functional.silu(x.float() @ Wg[0, c:c + step].float().T) * (x.float() @ Wu[0, c:c + step].float().T)
        assert float((a[:, c:c + step].float() - want).norm() / want.norm()) < 2.0 ** -8, c
