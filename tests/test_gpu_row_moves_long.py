"""Row moves of long rows: the combine with a workgroup per token (from 256 chunks of 16 bytes on; remainders of the chunks
per lane, K that four rows at a time do not divide) and the permute that moves x, xp or both past the 256 MB memory-side cache."""
import pytest

pytestmark = pytest.mark.gpu


def moves(N, H, K, dtype):
    import torch
    import paper_2605_05888_amd as hub
    print("row moves", N, H, K, dtype, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(N, H, generator=g, device="cuda").to(dtype)
    slot = torch.randperm(N * K, generator=torch.Generator().manual_seed(6)).to(torch.int32).cuda()
    row = torch.empty_like(slot)
    row[slot.long()] = torch.arange(N * K, dtype=torch.int32, device="cuda")
    xp = torch.full((N * K, H), 9.0, dtype=dtype, device="cuda")
    hub.moe_permute(x, K, slot, row, xp)
    assert torch.equal(xp[slot.long()].view(N, K, H), x[:, None].expand(N, K, H))
    return x, slot, xp, g


# bf16 / fp32 chunks: 255 | 256 | 257 | 511 | 512 | 1023 | 1025 | 1700; the last sizes of the one, the first of the other
@pytest.mark.parametrize("chunks", [255, 256, 257, 511, 512, 768, 1023, 1025, 1700])
@pytest.mark.parametrize("K,bf16", [(1, True), (2, False), (3, True), (4, False), (5, True), (8, True), (9, False)])
def test_long_rows(chunks, K, bf16):
    import torch
    import paper_2605_05888_amd as hub
    dtype = torch.bfloat16 if bf16 else torch.float32
    N, H = 5, chunks * (8 if bf16 else 4)
    x, slot, y, g = moves(N, H, K, dtype)
    y = torch.randn(N * K, H, generator=g, device="cuda").to(dtype)
    w = torch.rand(N, K, generator=g, device="cuda") / K
    out = torch.full((N, H), 9.0, dtype=dtype, device="cuda")
    hub.moe_combine(y, K, slot, w, out)
    rows = y[slot.long()].view(N, K, H).double()
    want = (rows * w[:, :, None].double()).sum(1)
    # K roundings of fp32 on partial sums of at most sum |w y|, then one rounding to bf16 (2^-9 of the value)
    bound = K * 2.0 ** -24 * (rows.abs() * w[:, :, None].double()).sum(1) + (2.0 ** -8 * want.abs() if bf16 else 0.0)
    assert bool(((out.double() - want).abs() <= bound + 1e-30).all())


# in MiB: xp 262, x 33 | x and xp 134 | xp 300, x 38 | x and xp 297 | xp 301 of short rows that share lines
@pytest.mark.parametrize("N,H,K", [(2100, 8200, 8), (8600, 8200, 1), (2400, 8200, 8), (19000, 8200, 1), (12000, 824, 16)])
def test_permute_past_the_cache(N, H, K):
    import torch
    moves(N, H, K, torch.bfloat16)
