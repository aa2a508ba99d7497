"""What MoELayerBuffers writes down about its buffers, as far as that shows without a GPU."""
import copy
import pickle

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


@pytest.mark.parametrize("again", [copy.copy, copy.deepcopy, lambda m: pickle.loads(pickle.dumps(m))])
def test_copies_start_without_plans(again):
    m = B.MoELayerBuffers(8, 64, 4, 2, 64, device="cpu")
    m._plans[2] = ("memory", 4096, [], [])
    c = again(m)
    assert c._plans == {} and m._plans[2][1] == 4096
    assert torch.equal(c.out, m.out) and c.k == 2
    c.out = torch.ones(8, 64)
    assert m._plans and not torch.equal(c.out, m.out)


def test_block_buffers_come_back_after_a_del():
    """The logits of the drop-in block are created where there are none: in a new layer, after a ``del``, and in a layer
    whose pickle predates them.  (The call itself is refused on host tensors.)"""
    m = B.MoELayerBuffers(8, 64, 4, 2, 64, device="cpu")
    x = torch.zeros(8, 64, dtype=torch.bfloat16)
    for _ in range(2):
        with pytest.raises(B.MoeError):
            m.run_block_fwd_bwd(x, torch.zeros(4, 64), x, m.dWg, m.dWu, m.dWd)
        assert m.logits.shape == (8, 4) and m.dlogits.shape == (8, 4) and m.dWr.shape == (4, 64)
        del m.logits


@pytest.mark.parametrize("form", ["plain", "gather", "fold"])
def test_input_is_kept_only_for_a_backward_that_reads_it(form, monkeypatch):
    m = B.MoELayerBuffers(8, 64, 4, 2, 64, device="cpu", gather=form == "gather", fold=form == "fold")
    ran = []
    monkeypatch.setattr(B.MoELayerBuffers, "_run", lambda self, *a: ran.append(a[1]))
    x = [torch.zeros(8, 64, dtype=torch.bfloat16) for _ in range(3)]
    w = m.dWg, m.dWu, m.dWd
    for step in (lambda: m.run_fwd(x[0], None, *w), lambda: m.run_fwd_bwd(x[1], None, x[0], *w),
                 lambda: m.run_block_fwd_bwd(x[2], None, x[0], *w)):
        step()
        m.run_bwd(x[0], *w)
        assert ran[-1] is (None if form == "plain" else ran[-2])
    # a pass that is refused leaves the input of the pass before
    def refuse(self, *a):
        raise B.MoeError("refused")
    monkeypatch.setattr(B.MoELayerBuffers, "_run", refuse)
    with pytest.raises(B.MoeError):
        m.run_fwd(x[0], None, *w)
    assert getattr(m, "_x", None) is (None if form == "plain" else x[2])
