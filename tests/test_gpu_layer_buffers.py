"""The layer's own buffers, checked once and written down for the native call: a buffer that is replaced, resized or taken
away afterwards counts as it would have at the first call."""
import struct

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


def _stage_calls(m, path, x, logits, dout, Wg, Wu, Wd):
    """What run_fwd_bwd does in one native call, through the calls of the single stages."""
    fold, plain = path == "fold", path == "plain"
    B.moe_route_permute(logits, x if plain else None, m.k, m.renormalize, m.e_begin, m.e_count, m.topk_idx, m.topk_w,
                        m.expert_offsets, m.row_token, m.slot_row, m.row_weight, m.xp, m.ws)
    if fold:
        B.moe_grouped_gemm_fwd_folded(x, m.row_token, m.row_weight, m.expert_offsets, Wg, Wu, Wd, m.g, m.u, m.h, m.yp)
        B.moe_unpermute_sum(m.yp, m.slot_row, m.out)
        B.moe_grouped_gemm_bwd_folded(dout, x, m.row_token, m.row_weight, m.slot_row, m.g, m.u, m.h, m.expert_offsets, Wg, Wu, Wd,
                                      m.dxp, m.dWg, m.dWu, m.dWd, m.dgate, m.ws)
    else:
        if plain:
            B.moe_grouped_gemm_fwd(m.xp, m.expert_offsets, Wg, Wu, Wd, m.g, m.u, m.h, m.yp)
        else:
            B.moe_grouped_gemm_fwd_gather(x, m.row_token, m.expert_offsets, Wg, Wu, Wd, m.g, m.u, m.h, m.yp)
        B.moe_unpermute_combine(m.yp, m.slot_row, m.topk_w, m.out)
        B.moe_unpermute_combine_bwd(dout, m.yp, m.slot_row, m.topk_w, m.dyp, m.dgate)
        if plain:
            B.moe_grouped_gemm_bwd(m.dyp, m.xp, m.g, m.u, m.h, m.expert_offsets, Wg, Wu, Wd, m.dxp, m.dWg, m.dWu, m.dWd, m.ws)
        else:
            B.moe_grouped_gemm_bwd_gather(m.dyp, x, m.row_token, m.g, m.u, m.h, m.expert_offsets, Wg, Wu, Wd, m.dxp, m.dWg, m.dWu,
                                          m.dWd, m.ws)
    B.moe_permute_bwd(m.dxp, m.slot_row, m.dx)


# tiled products with ragged tiles; streamed products of few rows; a rank's share; one whose expected rows are few, so that the
# number of rows decides on the device between the two (the stage calls, which know only T * k, take the tiled ones)
@pytest.mark.parametrize("T,d,E,k,f,eb,ec,hot", [
    (500, 192, 6, 3, 320, 0, 6, 0), (24, 320, 40, 4, 192, 0, 40, 0), (300, 128, 16, 4, 64, 4, 5, 0),
    (70, 320, 64, 4, 192, 8, 4, 0), (70, 320, 64, 4, 192, 8, 4, 30), (70, 320, 64, 4, 192, 8, 4, -30)])
@pytest.mark.parametrize("path", ["plain", "gather", "fold"])
def test_one_call_equals_the_stage_calls(path, T, d, E, k, f, eb, ec, hot):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(T)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    x, dout, logits = r(T, d).bfloat16(), r(T, d).bfloat16(), r(T, E)
    logits[:, eb:eb + ec] += hot
    w = [r(ec, *s).mul_(0.05).bfloat16() for s in ((f, d), (f, d), (d, f))]
    layers = [B.MoELayerBuffers(T, d, E, k, f, eb, ec, 1, gather=path == "gather", fold=path == "fold") for _ in range(2)]
    layers[0].run_fwd_bwd(x, logits, dout, *w)
    _stage_calls(layers[1], path, x, logits, dout, *w)
    one, stages = (m.results() for m in layers)
    rows = int(one["expert_offsets"][-1])
    if T == 70:
        assert rows == {0: rows, 30: T * k, -30: 0}[hot] and (rows <= 8 * ec) == (hot <= 0)
    for n, t in one.items():
        a, b = t, stages[n]
        if n in ("row_token", "row_weight", "xp", "g", "u", "h", "yp", "hw", "ypw", "dyp", "dxp"):     # T * k rows, not all local
            a, b = a[:rows], b[:rows]
        assert torch.equal(a, b), n


# The forward pass's combine and its backward in one kernel (run_fwd_bwd) against the two of run_fwd and run_bwd, and the gate
# gradient added up by the backward of the gather against the kernel of its own: rows of one to five groups of 64 pieces with
# a remainder, both sides of the rules on tokens (512, 2048), slots, bytes of rows (48 MB) and the share of local experts (a half),
# more slots than lanes
@pytest.mark.parametrize("T,d,E,k,eb,ec", [
    (513, 320, 12, 5, 0, 12), (40, 576, 12, 5, 3, 6), (600, 1088, 9, 3, 0, 9), (512, 1088, 9, 8, 0, 9), (33, 2112, 9, 1, 2, 4),
    (3100, 2112, 9, 4, 0, 9), (6000, 2112, 9, 4, 2, 3), (700, 2624, 9, 7, 0, 9), (20, 64, 90, 70, 5, 80),
    (2049, 576, 9, 1, 0, 9), (2049, 1088, 9, 2, 0, 9), (600, 1088, 9, 2, 0, 9), (600, 320, 9, 2, 0, 9)])
@pytest.mark.parametrize("path", ["plain", "gather", "fold"])
def test_both_passes_in_one_call(path, T, d, E, k, eb, ec):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(T + d)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    x, dout, logits, f = r(T, d).bfloat16(), r(T, d).bfloat16(), r(T, E), 64
    w = [r(ec, *s).mul_(0.05).bfloat16() for s in ((f, d), (f, d), (d, f))]
    one, two = (B.MoELayerBuffers(T, d, E, k, f, eb, ec, 1, gather=path == "gather", fold=path == "fold") for _ in range(2))
    one.run_fwd_bwd(x, logits, dout, *w)
    two.run_fwd(x, logits, *w)
    out = two.out.clone()
    apart = torch.empty_like(out)
    if path == "fold":
        B.moe_unpermute_sum(two.yp, two.slot_row, apart)
    else:
        B.moe_unpermute_combine(two.yp, two.slot_row, two.topk_w, apart)
    assert torch.equal(apart, out)
    if path == "fold":
        dx, dgate = torch.empty_like(two.dx), torch.empty_like(two.dgate)
        B.moe_grouped_gemm_bwd_folded(dout, x, two.row_token, two.row_weight, two.slot_row, two.g, two.u, two.h, two.expert_offsets, *w,
                                      two.dxp, two.dWg, two.dWu, two.dWd, dgate, two.ws)
        B.moe_permute_bwd(two.dxp, two.slot_row, dx)
    else:
        two.run_bwd(dout, *w)
        dx, dgate = two.dx, two.dgate
        rows = int(one.expert_offsets[-1])
        assert torch.equal(one.dyp[:rows], two.dyp[:rows])
    assert bool(torch.isfinite(out.float()).all()) and bool(torch.isfinite(dgate).all())
    assert torch.equal(one.out, out) and torch.equal(one.dgate, dgate) and torch.equal(one.dx, dx)
    assert torch.equal(one.dWd, two.dWd)


# A loss of half the squared output: the gradient handed in is the output buffer itself, read by the backward after the forward pass
# of the same call has written it (rows of one to five groups of 64 pieces, few and many tokens)
@pytest.mark.parametrize("T,d", [(600, 320), (40, 1088), (700, 2112)])
@pytest.mark.parametrize("path", ["plain", "gather", "fold"])
def test_the_output_as_its_own_gradient(path, T, d):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(T + d)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    E, k, f = 9, 4, 64
    x, logits = r(T, d).bfloat16(), r(T, E)
    w = [r(E, *s).mul_(0.05).bfloat16() for s in ((f, d), (f, d), (d, f))]
    one, two = (B.MoELayerBuffers(T, d, E, k, f, gather=path == "gather", fold=path == "fold") for _ in range(2))
    one.out.fill_(7.0)                       # what an earlier pass may have left there
    one.run_fwd_bwd(x, logits, one.out, *w)
    two.run_fwd(x, logits, *w)
    two.run_bwd(two.out, *w)
    for n in ("out", "dx", "dgate", "dWg", "dWu", "dWd"):
        assert torch.equal(getattr(one, n), getattr(two, n)), n


# Both passes in one call, a buffer that only the backward uses missing or misaligned: the call is refused, and the forward pass in
# front of it is complete (few and more than 64 slots)
@pytest.mark.parametrize("name", ["dout", "dyp", "dgate", "dxp", "dWd"])
@pytest.mark.parametrize("value", [0, 4])
@pytest.mark.parametrize("path,T,E,k", [("plain", 300, 9, 4), ("gather", 300, 9, 4), ("gather", 20, 90, 70), ("fold", 300, 9, 4)])
def test_a_refused_backward_leaves_the_forward_pass(path, T, E, k, name, value):
    if path == "fold" and name == "dyp":
        return                                      # not used there
    L, d, f = B.MoELayerBuffers, 1088, 64
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(T + k)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    x, dout, logits = r(T, d).bfloat16(), r(T, d).bfloat16(), r(T, E)
    w = [r(E, *s).mul_(0.05).bfloat16() for s in ((f, d), (f, d), (d, f))]
    m = L(T, d, E, k, f, gather=path == "gather", fold=path == "fold")
    m.run_fwd(x, logits, *w)
    want = m.out.clone()
    m.run_fwd_bwd(x, logits, dout, *w)
    blob, at = m._plans[L._FWD + L._BWD][:2]
    place = L._SIZES.size + (8 if name == "dout" else L._ARGS.size + 8 * L._ORDER.index(name))
    pointer = struct.unpack_from("=Q", blob, place)[0]
    struct.pack_into("=Q", blob, place, pointer + value if value else 0)
    m.out.fill_(7.0)
    assert B.load().moe_layer_run(at, L._FWD + L._BWD, B._stream()) == -1
    torch.cuda.synchronize()
    assert torch.equal(m.out, want)
