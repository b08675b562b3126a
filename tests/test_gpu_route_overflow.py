"""Selection where logits are not finite: fp32 sums of finite inputs that overflow to +-infinity or to NaN, and experts
masked by a bias of -infinity.  Every token gets K distinct experts of [0, E); NaN counts as -infinity, equal logits go to
the lower index; the other tokens are not touched, and moe_route_resolve_arrival draws rows inside its pointers only."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from layout_checks import check_layout_is_valid  # noqa: E402

# selection in the logits kernel (E <= 16) and one, two, four and sixteen experts per lane, with and without spare lanes
CASES = [(9, 8, 8, 2), (33, 8, 16, 16), (40, 12, 12, 5), (5, 8, 17, 3), (70, 8, 64, 6), (70, 16, 100, 8), (9, 8, 128, 32),
         (33, 8, 256, 8), (19, 8, 300, 7), (5, 8, 1024, 4), (8200, 8, 32, 4)]


@pytest.mark.parametrize("N,H,E,K", CASES)
def test_picks_are_distinct_experts_whatever_the_logits(N, H, E, K):
    import torch
    import gpu_layer as G
    import paper_2605_05888_amd as hub
    print("route, overflowed logits", N, H, E, K, flush=True)
    rng = np.random.default_rng(E * 37 + K)
    x = rng.standard_normal((N, H)).astype(np.float32)
    W = rng.standard_normal((H, E)).astype(np.float32)
    W[0], W[1] = rng.choice([-2.0, 0.0, 2.0], (2, E))
    W[2], W[3] = 2.0, -2.0
    kind = rng.integers(0, 5, N)                       # 0: an ordinary token
    kind[0] = 0
    x[kind == 1, 0] = 3e38                             # +inf, -inf and finite logits
    x[kind == 2, :2] = 3e38                            # ... and NaN (inf - inf)
    x[kind == 3, 0] = -3e38
    x[kind == 4, 2:4] = 3e38                           # NaN for every expert
    bias = rng.standard_normal(E).astype(np.float32)
    bias[rng.permutation(E)[:E - 1]] = -np.inf         # all experts but one masked
    for b in (None, bias):
        logits = oracle.logits(x, W, b)
        clean = np.where(np.isnan(logits), -np.inf, logits)
        want, _ = oracle.topk(clean, K, oracle.SOFTMAX_TOPK)
        assert np.isnan(logits[kind == 4]).all()
        picked = np.take_along_axis(logits, want.astype(np.int64), 1)
        usual = np.isfinite(picked).all(axis=1)        # (the weights of the others are NaN or not defined)
        dx, dW, db = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), None if b is None else torch.from_numpy(b).cuda()
        for mode in (oracle.SOFTMAX_TOPK, oracle.SIGMOID_TOPK):
            _, w_want = oracle.topk(clean, K, mode)
            idx, w, lg = G.gpu_route(dx, dW, db, K, mode)
            assert np.array_equal(G.host(lg), logits, equal_nan=True)
            assert np.array_equal(G.host(idx), want)
            assert np.max(np.abs(G.host(w).astype(np.float64) - w_want)[usual], initial=0.0) <= 2e-6
        # rows drawn on arrival: counts between guards, a valid packing of exactly these picks
        i32 = lambda n: torch.full((n,), -7, dtype=torch.int32, device="cuda")
        guarded = i32(E + 64)
        out = dict(expert_counts=guarded[32:32 + E], expert_offsets=i32(E + 1), dest_counts=i32(1), dest_offsets=i32(2),
                   slot_of_row=i32(N * K), row_of_slot=i32(N * K))
        idx2, w2 = torch.full((N, K), -1, dtype=torch.int32, device="cuda"), torch.zeros((N, K), device="cuda")
        hub.moe_route_resolve_arrival(dx, dW, db, K, 1, oracle.SIGMOID_TOPK, idx2, w2, *out.values(),
                                      torch.empty((N, E), device="cuda"))
        torch.cuda.synchronize()
        assert np.array_equal(G.host(idx2), want)
        assert (G.host(guarded[:32]) == -7).all() and (G.host(guarded[32 + E:]) == -7).all()
        check_layout_is_valid(want, E, 1, {k: G.host(v) for k, v in out.items()})


@pytest.mark.parametrize("N,H,E,bf16", [(19, 520, 30, False), (19, 584, 30, True), (40, 4, 6, False), (33, 1000, 15, True),
                                          (2100, 520, 32, False), (2100, 584, 32, True), (2100, 128, 32, True)])
def test_an_infinity_in_x_meets_the_columns_of_its_row_only(N, H, E, bf16):
    """H is no multiple of the 512 columns of a batch, or of the 128 of the large form's K tile: what stands for the columns
    past H must be neither an infinity of the row nor one of the next row."""
    import gpu_layer as G
    import moe_inputs as mi
    import moe_inputs.device as mid
    print("route, infinite x", N, H, E, bf16, flush=True)
    rng = np.random.default_rng(H + E)
    x = mi.f32_to_bf16_bits(rng.standard_normal((N, H)).astype(np.float32)) if bf16 else rng.standard_normal((N, H)).astype(np.float32)
    x[3, 1], x[8, 0], x[N - 1, 2] = (0x7F80, 0xFF80, 0x7F80) if bf16 else (np.inf, -np.inf, np.inf)
    W = rng.standard_normal((H, E)).astype(np.float32)
    want, _, logits = oracle.route(x, W, None, 2, oracle.SOFTMAX_TOPK)
    assert np.isinf(logits[[3, 8, N - 1]]).all() and np.isfinite(np.delete(logits, [3, 8, N - 1], 0)).all()
    idx, _, lg = G.gpu_route(mid.to_device(x), mid.to_device(W), None, 2, oracle.SOFTMAX_TOPK)
    assert np.array_equal(G.host(lg), logits)
    assert np.array_equal(G.host(idx), want)
