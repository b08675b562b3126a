"""The streams of a tile table: which tiles a workgroup finds where."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TABLE_MAGIC = 0x4D6F4554  # word 6 of a tile table's header


# full tiles of 256 rows, middle ones of up to 160, light ones of up to 64; (stream 0, stream 1, full, full and middle) in row tiles
@pytest.mark.parametrize("rows,want", [([600, 600, 600, 100, 160, 64], (11, 1, 9, 11)), # few light tiles: middle ones behind the full ones
                                       ([600, 600, 600, 100, 64, 1], (9, 3, 9, 10)),    # a sixth: with the light ones
                                       ([600, 161, 100, 160, 64, 1], (4, 4, 4, 6)),
                                       ([100, 65, 64, 1, 40], (0, 5, 0, 2)),           # no full tile: with the light ones
                                       ([320, 321, 512, 0], (5, 0, 5, 5)),
                                       ([300, 20, 10], (1, 2, 1, 1)),
                                       ([160, 160, 0], (0, 2, 0, 2))])
def test_streams_of_a_table(rows, want):
    import torch
    import paper_2605_05888_amd as hub
    print("streams", rows, flush=True)
    E, M, H, F = len(rows), sum(rows), 256, 640
    seg = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32, device="cuda")
    ws = torch.zeros(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F), dtype=torch.uint8, device="cuda")
    hub.moe_ffn_schedule(hub.BF16, M, H, F, seg, ws)
    words = ws.view(torch.int32).cpu().numpy()
    heads = [h for h in np.flatnonzero(words == TABLE_MAGIC) - 6 if h >= 0 and h % 64 == 0]
    assert len(heads) == 2
    for h, columns in zip(heads, (F // 128, H // 128)):   # (down projection: tiles of 128 columns)
        assert tuple(words[h:h + 4]) == tuple(columns * n for n in want)
