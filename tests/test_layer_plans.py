"""What MoELayerBuffers writes down about its buffers, as far as that shows without a GPU."""
import pytest
import torch

from paper_2604_00785_amd import binding as B


@pytest.mark.parametrize("change", [
    lambda t: t.t_(),                                              # other strides
    lambda t: t.resize_(t.shape[1], t.shape[0]),                   # other shape, still contiguous
    lambda t: setattr(t, "data", t.data.view(torch.int16)),        # other type at the same address
    lambda t: t.resize_(t.shape[0] - 1, t.shape[1]),
])
def test_in_place_changes_are_seen(change):
    ts = [torch.zeros(6, 4, dtype=torch.bfloat16), torch.zeros(6, 8, dtype=torch.bfloat16)]
    before = B.MoELayerBuffers._state(ts)
    assert B.MoELayerBuffers._state(ts) == before
    at = ts[1].data_ptr()
    change(ts[1])
    assert ts[1].data_ptr() == at
    assert B.MoELayerBuffers._state(ts) != before
