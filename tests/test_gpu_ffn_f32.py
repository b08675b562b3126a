"""fp32 expert FFN on the matrix cores (tiles of 32 rows x 64 columns, K tiles of 32): sizes on both sides of every edge,
against the fp64 oracle.  Bound: sums of n products in fp32 are off by at most n * 2^-24 relative to the sum of the
products' magnitudes; with two GEMMs of up to 100 terms of unit-variance results that is below 1e-5 in relative
L2 and below 1e-4 per element (the observed error is 3e-7)."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import moe_inputs as mi  # noqa: E402
import oracle  # noqa: E402

#        rows per expert,                                      H,  F
CASES = [([1], 4, 4),                                        # one row, one 16-byte chunk per row
         ([64, 0, 65, 63, 1, 128], 32, 64),                  # whole tiles, one row more, one row less
         ([5, 130, 0, 0, 7], 36, 68),                        # one chunk past a K tile and past a column tile
         ([31, 33, 97], 100, 60),                            # several K tiles, a ragged last one
         ([200], 28, 132),                                   # fewer columns than a K tile
         ([0] * 70 + [3, 0, 66] + [1] * 130, 64, 32)]        # more experts than lanes: several per lane


@pytest.mark.parametrize("gather", [False, True])
@pytest.mark.parametrize("rows,H,F", CASES)
def test_fp32_ffn_at_tile_edges(rows, H, F, gather):
    import torch
    import gpu_layer as G
    import moe_inputs.device as mid
    import paper_2605_05888_amd as hub
    E, M = len(rows), sum(rows)
    cfg = dataclasses.replace(mi.CONFIGS["tiny"], N=M, H=H, F=F, E=E, K=1, dtype=mi.F32, seed=91)
    print("fp32 ffn", rows[:8], H, F, gather, flush=True)
    seg = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    xp = mi.host_tensor(cfg, mi.STREAM_X)
    W = [mi.host_tensor(cfg, s) for s in (mi.STREAM_W_GATE, mi.STREAM_W_UP, mi.STREAM_W_DOWN)]
    want = oracle.ffn_rows(xp, seg, *W)
    dW, dseg = [mid.to_device(w) for w in W], mid.to_device(seg)
    if not gather:
        y = G.gpu_ffn(mid.to_device(xp), dseg, *dW)
    else:
        perm = np.random.default_rng(M).permutation(M).astype(np.int32)     # slot m holds row perm[m] of x
        x = np.empty_like(xp)
        x[perm] = xp
        ws = G.ws_tensor(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F, dtype=hub.F32))
        y = torch.zeros((M, H), dtype=torch.float32, device="cuda:0")
        hub.moe_ffn_schedule(hub.F32, M, H, F, dseg, ws)
        hub.moe_ffn_gate_up_gather(mid.to_device(x), 1, dseg, mid.to_device(perm), dW[0], dW[1], ws)
        hub.moe_ffn_down(dseg, dW[2], y, ws)
    torch.cuda.synchronize()
    G.check_close(G.host(y), want, 1e-4, 1e-5, what="fp32 ffn")


def test_more_tiles_than_one_grid_dimension_takes():
    """One row tile by 2^21 column tiles, eight row tiles to a band: 2^24 workgroups of 256 threads."""
    import torch
    import gpu_layer as G
    import paper_2605_05888_amd as hub
    M, H, F = 8, 4, 1 << 27
    print("fp32 ffn, many column tiles", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty(M, H, device="cuda").normal_(generator=g)
    Wg, Wu = (torch.empty(1, F, H, device="cuda").normal_(generator=g) for _ in range(2))
    seg = torch.tensor([0, M], dtype=torch.int32, device="cuda")
    ws = torch.full((hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=1, F=F, dtype=hub.F32) // 4,), float("nan"), device="cuda")
    hub.moe_ffn_gate_up(x, seg, Wg, Wu, ws)
    a = ws[:M * F].view(M, F)
    for lo in range(0, F, 1 << 23):
        part = slice(lo, lo + (1 << 23))
        want = torch.nn.functional.silu(x.double() @ Wg[0, part].double().T) * (x.double() @ Wu[0, part].double().T)
        # four products per sum: off by 2^-22 of their magnitudes at most, times the other factor
        assert float((a[:, part].double() - want).norm() / want.norm()) < 1e-6, lo


# Launches beyond 512 workgroups take fewer K tiles in flight (two in gate/up, three in down) and more workgroups per
# compute unit.  Workgroups, gate/up and down (row tiles rounded up to 8, times columns / 64, rounded up to 64):
MANY = [([313, 0, 97, 31, 300, 256, 33, 1, 480, 500, 499, 493], 516, 1028),   # 1920, 1024: ragged rows, columns and K
        ([300, 148], 2052, 2048),                                             # 512 (the last with more in flight), 576
        ([300, 148], 2048, 2052),                                             # 576, 512
        ([40] * 40, 100, 2500),                                               # 3840, 192: many experts, K shorter than the ring
        ([1500, 0, 0, 1], 4, 4096)]                                           # 3584 (one K tile of one chunk), 64


@pytest.mark.parametrize("gather", [False, True])
@pytest.mark.parametrize("rows,H,F", MANY, ids=[f"{sum(r)}-{h}-{f}" for r, h, f in MANY])
def test_fp32_ffn_of_many_workgroups(rows, H, F, gather):
    import torch
    import paper_2605_05888_amd as hub
    print("fp32 ffn, many workgroups", rows[:12], H, F, gather, flush=True)
    E, M = len(rows), sum(rows)
    seg = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(M)
    normal = lambda shape, std: torch.empty(shape, device="cuda").normal_(0.0, std, generator=g)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    dseg = torch.from_numpy(seg).cuda()
    ws = torch.full((hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F, dtype=hub.F32) // 4,), float("nan"), device="cuda")
    y = torch.full((M, H), float("nan"), device="cuda")
    if gather:
        perm = torch.randperm(M, generator=torch.Generator().manual_seed(5)).cuda()   # slot m holds row perm[m] of x
        x = torch.empty_like(xp)
        x[perm] = xp
        hub.moe_ffn_gate_up_gather(x, 1, dseg, perm.to(torch.int32), Wg, Wu, ws)
        hub.moe_ffn_down(dseg, Wd, y, ws)
    else:
        hub.moe_grouped_ffn(xp, dseg, Wg, Wu, Wd, y, ws)
    # n products of an fp32 sum are off by n * 2^-24 of their magnitudes at most, and as rounding errors mostly cancel by
    # some sqrt(n) * 2^-25 of the result: at n = 2500, twice, 3e-6
    for e, (lo, hi) in enumerate(zip(seg[:-1], seg[1:])):
        xe = xp[lo:hi].double()
        a = torch.nn.functional.silu(xe @ Wg[e].double().T) * (xe @ Wu[e].double().T)
        for got, want in ((ws[:M * F].view(M, F)[lo:hi], a), (y[lo:hi], a @ Wd[e].double().T)):
            assert lo == hi or float((got.double() - want).norm() / want.norm()) < 3e-6, e
