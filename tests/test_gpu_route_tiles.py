"""Router logits at the edges of its tiles: 16 tokens x 16 experts and batches of 512 columns in the small form,
32 tokens x 32 experts and K tiles of 128 columns in the large one (from 257 small tiles on, E % 4 == 0).
Bit for bit against the oracle's fp32 order; selection included."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import moe_inputs as mi  # noqa: E402
import oracle  # noqa: E402

CASES = [(1, 8, 16, 3, mi.BF16), (17, 520, 17, 5, mi.BF16), (16, 2048, 15, 15, mi.F32), (31, 2568, 33, 8, mi.BF16),
         (8192, 128, 16, 2, mi.BF16),                                    # selection in the logits kernel, many tiles
         (8160, 136, 20, 2, mi.BF16), (8193, 264, 20, 2, mi.F32),        # large form, ragged last tokens and columns
         (515, 8, 256, 8, mi.BF16), (2000, 648, 68, 4, mi.F32), (4100, 384, 32, 4, mi.BF16),
         (9001, 72, 100, 6, mi.BF16),                                    # several tiles per workgroup, one K tile each
         # large form, the tiles' list by experts (x smaller than W_r) and by tokens, in runs of different lengths per XCD
         (582, 136, 384, 2, mi.F32), (300, 264, 512, 8, mi.BF16), (129, 520, 1024, 4, mi.BF16), (1637, 72, 160, 1, mi.BF16),
         (2961, 264, 96, 3, mi.F32),
         # 256 tiles of the small form, 258 and 272
         (2048, 72, 32, 2, mi.BF16), (2049, 72, 32, 2, mi.BF16), (256, 136, 260, 3, mi.F32)]


@pytest.mark.parametrize("N,H,E,K,dtype", CASES)
def test_router_at_tile_edges(N, H, E, K, dtype):
    import gpu_layer as G
    import moe_inputs.device as mid
    cfg = dataclasses.replace(mi.CONFIGS["tiny"], N=N, H=H, E=E, K=K, dtype=dtype, seed=17)
    print("route tiles", N, H, E, K, dtype, flush=True)
    x, Wr = mi.host_tensor(cfg, mi.STREAM_X), mi.host_tensor(cfg, mi.STREAM_W_ROUTER)
    Wr[:, E - 1] = Wr[:, 0]                                              # first and last expert always tie
    bias = (np.arange(E) % 3 == 1).astype(np.float32) / 4
    bias[E - 1] = bias[0]
    for mode in (oracle.SOFTMAX_TOPK, oracle.SIGMOID_TOPK):
        o_idx, o_w, o_lg = oracle.route(x, Wr, bias, K, mode)
        idx, w, lg = G.gpu_route(mid.to_device(x), mid.to_device(Wr), mid.to_device(bias), K, mode)
        assert np.array_equal(G.host(lg).view(np.uint32), o_lg.view(np.uint32))
        assert np.array_equal(G.host(idx), o_idx)
        assert np.max(np.abs(G.host(w).astype(np.float64) - o_w)) <= 2e-6    # fp32 expf and one division
