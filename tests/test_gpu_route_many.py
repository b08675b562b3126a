"""Routing with more (token tile, expert tile) pairs than one dimension of a grid takes (2^23 workgroups of 512 threads):
the last tokens, which only the second row of the grid reaches, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402


def test_more_tiles_than_one_grid_dimension_takes():
    import torch
    import gpu_layer as G
    N, H, E, K, tail = 16 * 131080, 8, 1023, 2, 300      # 131080 x 64 tiles: 8 389 120 > 2^23; logits 8.6 GB
    print("route", N, H, E, K, flush=True)
    rng = np.random.default_rng(5)
    W, part = rng.standard_normal((H, E)).astype(np.float32), rng.standard_normal((4096, H)).astype(np.float32)
    x = torch.from_numpy(part).cuda().repeat(-(-N // 4096), 1)[:N].contiguous()
    idx, w, lg = G.gpu_route(x, torch.from_numpy(W).cuda(), None, K, oracle.SIGMOID_TOPK)
    want, w_want, logits = oracle.route(part, W, None, K, oracle.SIGMOID_TOPK)
    at = np.arange(N - tail, N) % 4096
    assert np.array_equal(G.host(lg[N - tail:]), logits[at])
    assert np.array_equal(G.host(idx[N - tail:]), want[at])
    # every token's picks: whole numbers, compared on the GPU
    full = torch.from_numpy(want).cuda().repeat(-(-N // 4096), 1)[:N]
    assert torch.equal(idx, full)
    assert np.max(np.abs(G.host(w[:4096]).astype(np.float64) - w_want)) <= 2e-6
