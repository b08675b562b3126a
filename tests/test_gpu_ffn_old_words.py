"""What earlier launches left in a workspace does not reach the next one: the words by which a workgroup's first thread hands
tiles to the others start over with every launch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TABLE_MAGIC = 0x4D6F4554                         # word 6 of a tile table's header
WORDS_BEFORE_TICKETS, TICKET_WORDS = 32, 8       # words 2, 3 of a workgroup's tickets: {tile, even sequence number}
OLD_TILE, OLD_SEQ = -2, 2                        # no tile, and one that no launch writes; the second draw's number


def old_words(ws):
    """Fills the workspace with {OLD_TILE, OLD_SEQ} pairs."""
    import torch
    ws.view(torch.int32)[0::2] = OLD_TILE
    ws.view(torch.int32)[1::2] = OLD_SEQ


def pairs(ws, groups):
    """The even pair of every workgroup, of both GEMMs' tables."""
    import torch
    words = ws.view(torch.int32).cpu().numpy()
    heads = [h for h in np.flatnonzero(words == TABLE_MAGIC) - 6 if h >= 0 and h % 64 == 0]
    assert len(heads) == 2
    return [words[h + WORDS_BEFORE_TICKETS:][:groups * TICKET_WORDS].reshape(groups, TICKET_WORDS)[:, 2:4] for h in heads]


# rows per expert: some workgroups get no tile | one tile each, one at a time | three and more, the next one fetched ahead
@pytest.mark.parametrize("E,H,F,rows", [(2, 512, 512, [300, 97]),
                                        (16, 1024, 2048, [64, 160, 40, 300]),
                                        (256, 1024, 1024, [1, 40, 64, 65, 97, 129, 160, 20])])
@pytest.mark.parametrize("one_launch", [False, True])
def test_old_words_in_the_workspace(E, H, F, rows, one_launch):
    import torch
    import paper_2605_05888_amd as hub
    print("old words", E, H, F, one_launch, flush=True)
    counts = (rows * E)[:E]
    M = sum(counts)
    seg = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(41)
    normal = lambda shape, std: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    xp, Wg, Wu, Wd = normal((M, H), 1.0), normal((E, F, H), H ** -0.5), normal((E, F, H), H ** -0.5), normal((E, H, F), F ** -0.5)
    ws = torch.zeros(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=F) // 8 * 8, dtype=torch.uint8, device="cuda")

    def ffn():
        y = torch.full((M, H), float("nan"), dtype=torch.bfloat16, device="cuda")
        hub.moe_ffn_schedule(hub.BF16, M, H, F, seg, ws)
        if one_launch:
            hub.moe_ffn_gate_up_down(xp, seg, Wg, Wu, Wd, y, ws)
        else:
            hub.moe_ffn_gate_up(xp, seg, Wg, Wu, ws)
            hub.moe_ffn_down(seg, Wd, y, ws)
        hub.moe_ffn_status(hub.BF16, M, H, F, E, ws)
        return y

    want = ffn()
    old_words(ws)
    assert torch.equal(ffn(), want)
    groups = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    for even in pairs(ws, groups):
        # every workgroup, also one that drew nothing, has put a number of this launch in place of the old one
        assert not (even == [OLD_TILE, OLD_SEQ]).all(axis=1).any()
    assert torch.equal(ffn(), want)
