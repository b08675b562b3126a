"""Address resolution by one workgroup (up to 8192 rows and some 900 experts) at the edges of its range, against the
oracle: whole numbers, exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402

CASES = [(1, 1, 1, 1), (1, 4, 7, 7), (3, 1, 64, 2), (511, 2, 2, 2), (1023, 1, 65, 5), (512, 2, 900, 9), (1025, 1, 33, 1),
         (341, 6, 256, 32), (683, 3, 909, 1), (683, 3, 910, 2), (513, 4, 128, 8), (4095, 1, 16, 4), (1365, 3, 12, 3),
         (4097, 1, 1, 1), (2731, 3, 48, 6), (8191, 1, 1000, 8), (1024, 8, 256, 32), (8193, 1, 8, 2)]


@pytest.mark.parametrize("skewed", [False, True])
@pytest.mark.parametrize("N,K,E,G", CASES)
def test_layout_at_the_edges(N, K, E, G, skewed):
    import gpu_layer as GL
    import moe_inputs.device as mid
    print("layout", N, K, E, G, skewed, flush=True)
    rng = np.random.default_rng(N * 31 + E)
    if skewed: # token after token the same experts, and most of the others get nothing
        idx = np.tile(rng.permutation(E)[:K], (N, 1))
        idx[::7] = rng.permutation(E)[:K]
    else:
        idx = np.argsort(rng.random((N, E)), axis=1)[:, :K]
    idx = np.ascontiguousarray(idx, dtype=np.int32)
    got, want = GL.gpu_layout(mid.to_device(idx), E, G), oracle.layout(idx, E, G)
    for k in want:
        assert np.array_equal(GL.host(got[k]), want[k]), k
