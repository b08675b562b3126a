"""Down projection into rows so wide that those of one tile take more than 4 GiB, more than the byte count that bounds its stores
can hold."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,H", [(330, 64 * 105469),    # a full row tile and one of 74 rows; 318 rows fit into 4 GiB
                                 (320, 64 * 105469),    # a tall tile with two block rows more
                                 (288, 64 * 116600),    # one block row more
                                 (300, 64 * 131073)])   # 256 rows do not fit
def test_rows_of_13_megabytes(M, H):
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
