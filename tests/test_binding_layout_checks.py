"""The checks of the layout calls' six arrays: what is passed on, and the exception that names the first wrong one (no GPU needed)."""
import types

import pytest
import torch

from paper_2605_05888_amd import binding

NAMES = ("expert_counts", "expert_offsets", "dest_counts", "dest_offsets", "slot_of_row", "row_of_slot")
SIZES = (8, 9, 2, 3, 40, 40)


def arrays(**wrong):
    def one(name, n):
        a = dict(dtype=torch.int32, cuda=True, dense=True, n=n)
        a.update(wrong.get(name, {}))
        return types.SimpleNamespace(dtype=a["dtype"], is_cuda=a["cuda"], is_contiguous=lambda: a["dense"], numel=lambda: a["n"])
    return [one(name, n) for name, n in zip(NAMES, SIZES)]


def test_right_arrays_pass():
    assert binding._need_layout(8, 2, 40, *arrays()) is None


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("wrong,error", [({"dtype": torch.int64}, TypeError), ({"cuda": False}, TypeError),
                                         ({"dense": False}, TypeError), ({"n": 7}, AssertionError)])
def test_a_wrong_array_is_named(name, wrong, error):
    with pytest.raises(error, match=name):
        binding._need_layout(8, 2, 40, *arrays(**{name: wrong}))
