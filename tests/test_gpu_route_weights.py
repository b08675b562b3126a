"""Normalisation of the selected scores: summed in fp32 by rank, in pairs 16, 8, 4, 2, 1 apart, whichever kernel selects
(E <= 16: the logits kernel), so that moe_route and moe_route_resolve_arrival give the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402

CASES = [(3, 3), (12, 3), (12, 7), (16, 4), (16, 8), (16, 16), (17, 8), (64, 12), (100, 17), (40, 32), (256, 24)]


def pair_sum(s, n):
    """s [T, n] fp32: additions of neighbours n/2, n/4, ... 1 apart."""
    while n > 1:
        n //= 2
        s = (s[:, :n] + s[:, n:2 * n]).astype(np.float32)
    return s[:, 0]


@pytest.mark.parametrize("E,K", CASES)
def test_scores_are_summed_by_rank(E, K):
    import gpu_layer as G
    import moe_inputs.device as mid
    print("route weights", E, K, flush=True)
    T = 256
    rng = np.random.default_rng(E + K)
    # one score of 1 and others below half a unit in the last place of it: what a sum drops depends on its order.
    # x picks one row of W_r, so the logits are its numbers exactly.
    W = rng.uniform(-17.6, -15.5, (T, E)).astype(np.float32)
    W[np.arange(T), rng.integers(0, E, T)] = 0.0
    x = np.eye(T, dtype=np.float32)
    idx, w, lg = G.gpu_route(mid.to_device(x), mid.to_device(W), None, K, oracle.SOFTMAX_TOPK)
    assert np.array_equal(G.host(lg), W)
    order = np.argsort(-W, axis=1, kind="stable")[:, :K]
    assert np.array_equal(G.host(idx), order)
    exact = np.exp(np.take_along_axis(W, order, 1).astype(np.float64))

    def summed(rel, by_position=False):
        s = np.zeros((T, 32), np.float32)
        t = np.where(exact == 1.0, 1.0, exact * (1.0 + rel)).astype(np.float32)
        if by_position:
            np.put_along_axis(s, order, t, 1)
            return pair_sum(s[:, :16], 16)
        s[:, :K] = t
        return pair_sum(s, 32)

    want = summed(0.0)
    # the device's expf may differ in the last bits of a score: tokens where that decides nothing
    sure = (summed(1e-6) == want) & (summed(-1e-6) == want)
    assert sure.sum() > T // 2
    assert np.array_equal(G.host(w)[sure, 0], (np.float32(1.0) / want)[sure])
    if E <= 16:
        assert (summed(0.0, True) != want)[sure].any()  # (the order by expert would be told apart)


@pytest.mark.parametrize("mode", [oracle.SOFTMAX_TOPK, oracle.SIGMOID_TOPK])
@pytest.mark.parametrize("E,K", CASES)
def test_both_routing_calls_give_the_same_weights(E, K, mode):
    import gpu_layer as G
    import moe_inputs.device as mid
    print("route weights, both calls", E, K, mode, flush=True)
    rng = np.random.default_rng(E * 33 + K)
    x, W = rng.standard_normal((300, 64)).astype(np.float32), rng.standard_normal((64, E)).astype(np.float32) / 4
    dx, dW, db = mid.to_device(x), mid.to_device(W), mid.to_device(rng.standard_normal(E).astype(np.float32))
    idx, w, _ = G.gpu_route(dx, dW, db, K, mode)
    idx2, w2, _, _ = G.gpu_route_resolve_arrival(dx, dW, db, K, 1, mode)
    assert np.array_equal(G.host(idx), G.host(idx2))
    assert np.array_equal(G.host(w).view(np.uint32), G.host(w2).view(np.uint32))
