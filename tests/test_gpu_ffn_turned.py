"""Reductions that start past the first column and wrap around (rows of the weights a multiple of 4 KiB apart, up to 8192
columns), in every form of tile: shallow, of 160 rows, ragged, full, tall by a shared and by an own block row, several row tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS = [300, 20, 64, 65, 276, 1, 0, 530]
BLOCKS = [97, 129, 160, 161, 256]  # tiles of 160 rows with four and five block rows, single tiles of 256
# H, F, how often ROWS (reductions are turned from 192 column tiles on, of all experts together)
SIZES = [(2048, 128 * 17 + 64, 1),  # too few tiles: not turned
         (2048, 128 * 17 + 64, 2),  # gate/up turned: shallow tiles at 0 and 1 K tiles of 16, others from column tile 8 on
         (256 * 17 + 64, 2048, 1),  # down projection turned
         (4096, 4096, 1),           # both, four starting points
         (6144, 1216, 1),
         (6144, 1216, 4)]           # a number of K tiles that 16 does not divide evenly into turns


@pytest.mark.parametrize("H,F,times,more", [(*size, []) for size in SIZES] + [(4096, 4096, 1, BLOCKS)])
def test_turned_reduction(H, F, times, more):
    import torch
    import paper_2605_05888_amd as hub
    print("turned", H, F, times, len(more), flush=True)
    rows_of = ROWS * times + more
    E, M = len(rows_of), sum(rows_of)
    seg = np.concatenate([[0], np.cumsum(rows_of)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(11)
    normal = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    dseg = torch.from_numpy(seg).cuda()
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hub.moe_grouped_ffn(xp, dseg, Wg, Wu, Wd, y, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
    for e in range(E):
        lo, hi = int(seg[e]), int(seg[e + 1])
        if lo == hi:
            continue
        x = xp[lo:hi].double()
        a = torch.nn.functional.silu(x @ Wg[e].double().T) * (x @ Wu[e].double().T)
        want = a.to(torch.bfloat16).double() @ Wd[e].double().T
        # one rounding of y (2^-9 at most); bf16 steps of `a` that fall on the other side are far rarer than that
        assert float((y[lo:hi].double() - want).norm() / want.norm()) < 2.0 ** -9, e
    # rows fetched through a map: bit for bit the same
    perm = torch.randperm(M, generator=torch.Generator().manual_seed(3)).cuda()
    x = torch.empty_like(xp)
    x[perm] = xp
    y2 = torch.full_like(y, float("nan"))
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_gather(x, 1, dseg, perm.to(torch.int32), Wg, Wu, ws)
    hub.moe_ffn_down(dseg, Wd, y2, ws)
    assert torch.equal(y, y2)


# narrow column tiles in the down projection (up to 256 tiles of 256 columns) and wide ones; gate/up, down or both turned
FORMS = [(2048, 320, 1), (320, 2048, 1), (2048, 4096, 1), (6144, 1216, 1), (5696, 2048, 1), (6144, 4096, 1),
         (2048, 320, 8), (320, 2048, 8), (2048, 4096, 2), (6144, 1216, 4), (5696, 2048, 2)]


@pytest.mark.parametrize("H,F,times,more", [(*form, []) for form in FORMS] +
                         [(2048, 320, 8, BLOCKS), (320, 2048, 8, BLOCKS),   # gate/up, narrow down projection turned
                          (6144, 4096, 1, BLOCKS)])                         # both
def test_turned_reduction_in_the_other_forms(H, F, times, more):
    """Both GEMMs in one launch, the combine in the down projection's epilogue, and every segment reversed (so that a
    remainder of rows that rode with a full tile is an ordinary part of it): the bits of the separate launches."""
    import torch
    import paper_2605_05888_amd as hub
    print("turned, other forms", H, F, times, len(more), flush=True)
    rows_of = ROWS * times + more
    E, M = len(rows_of), sum(rows_of)
    seg = np.concatenate([[0], np.cumsum(rows_of)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(12)
    normal = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    dseg = torch.from_numpy(seg).cuda()
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hub.moe_grouped_ffn(xp, dseg, Wg, Wu, Wd, y, ws)
    want = torch.cat([(torch.nn.functional.silu(x @ Wg[e].double().T) * (x @ Wu[e].double().T)).to(torch.bfloat16).double() @
                      Wd[e].double().T for e, x in enumerate(xp[lo:hi].double() for lo, hi in zip(seg[:-1], seg[1:]))])
    assert float((y.double() - want).norm() / want.norm()) < 2.0 ** -9   # (one rounding of y)

    def one_launch(rows, times):
        out = torch.full_like(y, float("nan"))
        hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
        for _ in range(times):
            hub.moe_ffn_gate_up_down(rows, dseg, Wg, Wu, Wd, out, ws)
        hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
        return out

    assert torch.equal(one_launch(xp, 1), y)
    assert torch.equal(one_launch(xp, 3), y)                             # three times over one schedule
    rev = torch.cat([torch.arange(lo, hi).flip(0) for lo, hi in zip(seg[:-1], seg[1:])]).cuda()
    y_rev = torch.full_like(y, float("nan"))
    hub.moe_grouped_ffn(xp[rev].contiguous(), dseg, Wg, Wu, Wd, y_rev, ws)
    assert torch.equal(y_rev, y[rev])
    assert torch.equal(one_launch(xp[rev].contiguous(), 1), y[rev])
    # rows fetched through the map, and added to their tokens' sums (top-1, weight 2: exact doubles); x[rev[m]] is row m
    x = torch.empty_like(xp)
    x[rev] = xp
    rows = rev.to(torch.int32)
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_gather(x, 1, dseg, rows, Wg, Wu, ws)
    sums, out = torch.empty(M, H, device="cuda"), torch.empty(M, H, dtype=torch.bfloat16, device="cuda")
    hub.moe_ffn_down_combine(1, dseg, Wd, rows, torch.full((M, 1), 2.0, device="cuda"), sums, out, ws)
    assert torch.equal(out[rev], (2.0 * y.float()).to(torch.bfloat16))
