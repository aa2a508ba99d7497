"""The layer's own buffers, checked once and written down for the native call: a buffer that is replaced, resized or taken
away afterwards counts as it would have at the first call."""
import pytest
import torch

from paper_2604_00785_amd import binding as B
from paper_2604_00785_amd import workloads as W

pytestmark = pytest.mark.gpu


def _layer(path):
    cfg = W.CONFIGS["tiny"]
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    a = {"x": r(cfg.T, cfg.d).bfloat16(), "dout": r(cfg.T, cfg.d).bfloat16(), "logits": r(cfg.T, cfg.E)}
    w = [r(cfg.n_local, *s).mul_(0.02).bfloat16() for s in ((cfg.f, cfg.d), (cfg.f, cfg.d), (cfg.d, cfg.f))]
    m = B.MoELayerBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.f, cfg.e_begin, cfg.n_local, cfg.renormalize,
                          gather=path == "gather", fold=path == "fold")
    return m, a, w


@pytest.mark.parametrize("path", ["plain", "gather", "fold"])
def test_replaced_buffers(path):
    m, a, w = _layer(path)
    step = lambda: m.run_fwd_bwd(a["x"], a["logits"], a["dout"], *w)
    step()
    want = {n: getattr(m, n).clone() for n in ("out", "dx", "dgate", "dWg", "dWu", "dWd")}
    # refused, though the address is the same: a smaller view, another type; a buffer resized in place
    for name in ("g", "dxp", "topk_idx", "out"):
        t = getattr(m, name)
        for bad in (t[:-1], t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.float32)):
            setattr(m, name, bad)
            with pytest.raises(B.MoeError):
                step()
        setattr(m, name, t)
    shape = m.h.shape
    m.h.resize_(shape[0] - 1, shape[1])
    with pytest.raises(B.MoeError):
        step()
    m.h.resize_(shape)
    # refused, though address and element count are the same: other strides, another shape
    for name in ("out", "dxp", "topk_w"):
        t = getattr(m, name)
        shape = t.shape
        t.t_()
        with pytest.raises(B.MoeError):
            step()
        t.t_()
        t.resize_(shape[1], shape[0])
        with pytest.raises(B.MoeError):
            step()
        t.resize_(shape)
    # a new buffer is the one that is written
    old = m.out
    old.fill_(7.0)
    m.out = torch.zeros_like(old)
    step()
    assert bool((old == 7.0).all())
    for n, t in want.items():
        assert torch.equal(getattr(m, n), t), n
    # a forward pass alone does without the buffers of the backward pass
    for n in ("dyp", "dxp", "dx", "dgate", "dWg", "dWu", "dWd"):
        setattr(m, n, None)
    m.out.zero_()
    m.run_fwd(a["x"], a["logits"], *w)
    assert torch.equal(m.out, want["out"])


@pytest.mark.parametrize("path", ["plain", "gather", "fold"])
def test_wider_arguments(path):
    """x may lie in front of other rows, and the logits may have columns that the layer was not laid out for, where no other
    buffer has to match them; fewer rows of x than tokens are refused."""
    m, a, w = _layer(path)
    m.run_fwd(a["x"], a["logits"], *w)
    want = {n: getattr(m, n).clone() for n in ("topk_idx", "topk_w", "out")}
    longer = torch.cat([a["x"], torch.full_like(a["x"][:5], float("nan"))])
    wider = torch.cat([a["logits"], torch.full_like(a["logits"][:, :3], -1e30)], 1)
    m.out.zero_()
    m.run_fwd(longer, wider, *w)
    for n, t in want.items():
        assert torch.equal(getattr(m, n), t), n
    if path == "fold":                   # its backward reads dout by the token too, and wants both of one size
        with pytest.raises(B.MoeError):
            m.run_bwd(a["dout"], *w)
    else:
        m.run_fwd_bwd(a["x"], a["logits"], a["dout"], *w)
        grads = {n: getattr(m, n).clone() for n in ("dx", "dgate", "dWg", "dWu", "dWd")}
        m.run_fwd_bwd(longer, wider, a["dout"], *w)
        for n, t in grads.items():
            assert torch.equal(getattr(m, n), t), n
    for x, lg in ((a["x"][:-1], a["logits"]), (longer[:, :-8].contiguous(), a["logits"]), (a["x"], a["logits"][:-1]), (a["x"][0], a["logits"])):
        with pytest.raises(B.MoeError):
            m.run_fwd(x, lg, *w)
    with pytest.raises(B.MoeError):
        m.run_block_fwd_bwd(longer, torch.zeros(m.E, m.d, device="cuda:0"), a["dout"], *w)
