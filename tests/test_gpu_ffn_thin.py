"""The expert FFN's form for few rows (csrc/ffn_thin.hip) and the rule that picks it, against float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# H and F in K lines of 64 columns: one, fewer than the wavefronts, a remainder over the turns, and enough columns for
# the wide form (more than 4 rows per expert, E * F / 32 and E * H / 64 at least 384)
CASES = [
    # rows per expert, H, F
    ([1], 64, 64),
    ([0, 1, 0, 15], 192, 128),
    ([3, 0, 13, 16], 320, 576),
    ([16, 17, 32, 1, 0, 30], 448, 64),          # M > 16: blocks of 16, 32 and 64 rows in one launch
    ([33, 64, 2, 0, 1], 128, 1088),
    ([65, 0, 1, 62, 0, 0, 0, 0], 576, 320),     # an expert with two row tiles
    ([200] + [0] * 12 + [8, 1, 0], 256, 192),   # most rows with one expert
    ([5] * 16, 1536, 896),                      # wide tiles in both GEMMs
    ([64] + [0] * 30 + [1], 832, 448),          # wide tiles, row blocks of four
    ([32] * 8, 256, 256),                       # the rule's last rows ...
    ([33] * 8, 256, 256),                       # ... and the tiled kernel
    ([16] * 16, 4096 + 64, 256),                # down projection tiled (more column tiles than the rule takes)
    ([4] * 8, 64, 128 * 28),                    # most column tiles with a few rows ...
    ([5] * 8, 64, 128 * 28),                    # ... and short reductions
]


@pytest.mark.parametrize("rows,H,F", CASES, ids=[f"{len(r)}x{max(r)}-{h}-{f}" for r, h, f in CASES])
def test_few_rows(rows, H, F):
    import torch
    import paper_2605_05888_amd as hub
    print("few rows", rows, H, F, flush=True)
    E, M = len(rows), sum(rows)
    seg = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    g = torch.Generator().manual_seed(7)
    normal = lambda shape, std: (torch.randn(shape, generator=g) * std).to(torch.bfloat16)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    want = torch.zeros(M, H, dtype=torch.float64)
    for e in range(E):
        x = xp[seg[e]:seg[e + 1]].double()
        a = torch.nn.functional.silu(x @ Wg[e].double().T) * (x @ Wu[e].double().T)
        want[seg[e]:seg[e + 1]] = a.to(torch.bfloat16).double() @ Wd[e].double().T
    dev = lambda t: t.cuda()
    dx, dg, du, dd, dseg = dev(xp), dev(Wg), dev(Wu), dev(Wd), dev(torch.from_numpy(seg))
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hub.moe_grouped_ffn(dx, dseg, dg, du, dd, y, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
    got = y.cpu().double()
    # one rounding of y (2^-9 at most), and the bf16 steps of `a` that fp32 and fp64 sums round to different sides:
    # one in about sqrt(H) * 2^-24 / 2^-9 of its elements, far below the first
    assert torch.isfinite(got).all()
    assert float((got - want).norm() / want.norm()) < 2.0 ** -9
    # rows fetched from x through a map, top-1: bit for bit the same
    perm = torch.randperm(M, generator=g)
    x = torch.empty_like(xp)
    x[perm] = xp
    y2 = torch.full_like(y, float("nan"))
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_gather(dev(x), 1, dseg, dev(perm.to(torch.int32)), dg, du, ws)
    hub.moe_ffn_down(dseg, dd, y2, ws)
    assert torch.equal(y, y2)
    # ... both GEMMs in one call, and the down projection with the combine in it (top-1, weight 2: exact doubles)
    y3 = torch.full_like(y, float("nan"))
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_down(dx, dseg, dg, du, dd, y3, ws)
    assert torch.equal(y, y3)
    sums, out = torch.empty(M, H, device="cuda"), torch.empty(M, H, dtype=torch.bfloat16, device="cuda")
    weight = torch.full((M, 1), 2.0, device="cuda")
    hub.moe_ffn_down_combine(1, dseg, dd, dev(perm.to(torch.int32)), weight, sums, out, ws)
    assert torch.equal(out.cpu()[perm], (2.0 * y.float()).to(torch.bfloat16).cpu())


def test_few_rows_need_their_schedule():
    import torch
    import paper_2605_05888_amd as hub
    M, H, F, E = 4, 128, 128, 4
    ws = torch.zeros(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    w = torch.zeros(E, F, H, dtype=torch.bfloat16, device="cuda")
    seg = torch.arange(E + 1, dtype=torch.int32, device="cuda")
    hub.moe_ffn_gate_up(torch.zeros(M, H, dtype=torch.bfloat16, device="cuda"), seg, w, w, ws)
    with pytest.raises(hub.MoEHubError, match="MOE_ERR_STATE"):
        hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)


# tokens, experts, top-K, H, F: the down projection thin or tiled, one row per expert up to whole row blocks
@pytest.mark.parametrize("N,E,K,H,F", [(1, 64, 4, 2048, 1408), (1, 4, 4, 512, 256), (3, 8, 2, 320, 576), (40, 16, 3, 256, 192),
                                       (64, 8, 4, 448, 320)])
def test_few_tokens_with_several_experts_each(N, E, K, H, F):
    """Rows fetched from x through a map with K slots per token: the bits of permute and the plain form; the down
    projection that adds K weighted rows per token against float64."""
    import torch
    import paper_2605_05888_amd as hub
    print("few tokens", N, E, K, H, F, flush=True)
    g = torch.Generator().manual_seed(N + E)
    normal = lambda shape, std: (torch.randn(shape, generator=g) * std).to(torch.bfloat16).cuda()
    x, Wg, Wu, Wd = normal((N, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    idx = torch.stack([torch.randperm(E, generator=g)[:K] for _ in range(N)]).to(torch.int32).cuda()
    w = torch.rand((N, K), generator=g).cuda() + 0.5
    M = N * K
    i32 = lambda n: torch.empty(n, dtype=torch.int32, device="cuda")
    raw = lambda n: torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    counts, offsets, dest, dest_off, slot, row = i32(E), i32(E + 1), i32(1), i32(2), i32(M), i32(M)
    hub.moe_dispatch_layout(idx, E, 1, counts, offsets, dest, dest_off, slot, row,
                            raw(hub.workspace_bytes(hub.OP_DISPATCH_LAYOUT, N=N, E=E, K=K)))
    xp, y, y2 = x.new_empty(M, H), x.new_full((M, H), float("nan")), x.new_full((M, H), float("nan"))
    ws = raw(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F))
    hub.moe_permute(x, K, slot, row, xp)
    hub.moe_grouped_ffn(xp, offsets, Wg, Wu, Wd, y, ws)
    hub.moe_ffn_schedule(hub.BF16, M, H, F, offsets, ws)
    hub.moe_ffn_gate_up_gather(x, K, offsets, row, Wg, Wu, ws)
    hub.moe_ffn_down(offsets, Wd, y2, ws)
    assert torch.equal(y, y2)
    sums, out = torch.empty(N, H, device="cuda"), x.new_empty(N, H)
    hub.moe_ffn_down_combine(K, offsets, Wd, row, w, sums, out, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
    want_y, want = torch.zeros(M, H, dtype=torch.float64, device="cuda"), torch.zeros(N, H, dtype=torch.float64, device="cuda")
    for n in range(N):
        for k in range(K):
            e, xr = int(idx[n, k]), x[n].double()
            a = torch.nn.functional.silu(Wg[e].double() @ xr) * (Wu[e].double() @ xr)
            want_y[slot[n * K + k]] = Wd[e].double() @ a.to(torch.bfloat16).double()
            want[n] += float(w[n, k]) * want_y[slot[n * K + k]]
    # one rounding to bf16 each (2^-9 at most); fp32 sums are far below that
    assert float((y.double() - want_y).norm() / want_y.norm()) < 2.0 ** -9
    assert float((out.double() - want).norm() / want.norm()) < 2.0 ** -9


# On both sides of the rule's lines: tiles (gate/up: of 128 columns; down: of 128, or of 256 beyond 256 of those), rows per
# expert, reduction length.
EDGES = [
    ([30, 31, 34, 33], 6144, 2176),      # gate/up 68 tiles, 128 rows * 6144 (24 * 8192 per expert): tiled
    ([30, 31, 34, 32], 6144, 2176),      # ... and the last few-row launch
    ([1, 4, 7, 4], 6080, 4224),          # 132 tiles, 16 rows * 6080 ...
    ([1, 4, 7, 4], 6144, 4224),          # ... and one K tile more
    ([4, 0, 8, 4], 4096, 5760),          # 180 tiles, K 4096 ...
    ([4, 0, 8, 4], 4160, 5760),          # ... and one K tile more
    ([4, 0, 8, 4], 5760, 4096),          # down projection of 180 narrow tiles, K 4096 ...
    ([4, 0, 8, 4], 5760, 4160),          # ... and one K tile more
    ([16, 9, 23, 16], 1024, 12416),      # gate/up 388 tiles: K 1024 with 16 rows ...
    ([16, 9, 23, 16], 1088, 12416),      # ... 1088 with 16 (tiled) ...
    ([2, 1, 3, 2], 1088, 12416),         # ... and with 2
    ([16, 9, 23, 16], 1088, 12288),      # 384 tiles
]


@pytest.mark.parametrize("rows,H,F", EDGES, ids=[f"{len(r)}x{max(r)}-{h}-{f}" for r, h, f in EDGES])
def test_lines_of_the_rule(rows, H, F):
    import torch
    import paper_2605_05888_amd as hub
    print("few rows, lines of the rule", rows, H, F, flush=True)
    E, M = len(rows), sum(rows)
    seg = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(17)
    normal = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    dseg = torch.from_numpy(seg).cuda()
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    hub.moe_grouped_ffn(xp, dseg, Wg, Wu, Wd, y, ws)
    hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
    y2 = torch.full_like(y, float("nan"))
    hub.moe_ffn_schedule(hub.BF16, M, H, F, dseg, ws)
    hub.moe_ffn_gate_up_down(xp, dseg, Wg, Wu, Wd, y2, ws)
    assert torch.equal(y, y2)
    for e in range(E):
        lo, hi = int(seg[e]), int(seg[e + 1])
        if lo == hi:
            continue
        x = xp[lo:hi].double()
        a = torch.nn.functional.silu(x @ Wg[e].double().T) * (x @ Wu[e].double().T)
        want = a.to(torch.bfloat16).double() @ Wd[e].double().T
        assert float((y[lo:hi].double() - want).norm() / want.norm()) < 2.0 ** -9, e   # (one rounding of y)


@pytest.mark.parametrize("H,F,E,M", [(2048, 1408, 8, 100), (2048, 2048, 24, 800), (576, 320, 6, 500)], ids=["few-rows", "turned", "tiled"])
def test_a_row_does_not_depend_on_the_others(H, F, E, M):
    """Same launch size, other rows and other segments (on the same side of 64 rows): a row keeps its bits."""
    import torch
    import paper_2605_05888_amd as hub
    print("row by itself", H, F, E, M, flush=True)
    g = torch.Generator(device="cuda").manual_seed(29)
    normal = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    Wg, Wu, Wd = normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    ws = torch.empty(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    small, large = normal((5, H), 1.0), normal((70, H), 1.0)

    def rows_of(n_small, n_large, at):
        seg = [0, n_small, n_small + n_large] + [M] * (E - 2)   # expert 2 takes the rest
        x = normal((M, H), 1.0)
        x[at:at + 5] = small
        x[n_small:n_small + 70] = large
        y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
        hub.moe_grouped_ffn(x, torch.tensor(seg, dtype=torch.int32, device="cuda"), Wg, Wu, Wd, y, ws)
        hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
        return y[at:at + 5], y[n_small:n_small + 70]

    a, b = rows_of(5, 70, 0), rows_of(23, 72, 17)
    assert torch.isfinite(a[0]).all() and torch.isfinite(a[1]).all()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
