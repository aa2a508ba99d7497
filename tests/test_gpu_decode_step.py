"""The forward pass of a few tokens, whose layer call takes kernels that do several stages each: the bits of the stages one by one.
Sizes on both sides of what those kernels take: 64 pairs, 8 tokens, ten winners of a wave one after the other, 4 tokens and 8
slots for down with the combine, one expert, shares of the experts, odd numbers of column tiles, reductions of any length."""
import pytest
import torch

import test_gpu_layer_buffers as L
from paper_2604_00785_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,d,E,k,f,eb,ec,renorm", [
    (1, 2048, 64, 8, 1024, 0, 64, 1),
    (2, 2048, 64, 8, 2048, 0, 64, 1),         # reductions that begin at a step of the expert's in both products
    (4, 1088, 96, 8, 576, 0, 96, 0),          # two passes of four tokens; the last call of down with the combine
    (5, 1088, 96, 8, 576, 0, 96, 1),          # ... the first without
    (4, 576, 20, 9, 192, 0, 20, 1),           # nine slots: not in one kernel
    (3, 64, 5, 5, 64, 1, 3, 0),               # a share, one step per reduction, four column tiles
    (4, 320, 8, 1, 448, 0, 8, 1),
    (1, 192, 1, 1, 128, 0, 1, 1),             # one expert
    (16, 256, 8, 4, 128, 0, 8, 1),            # 64 pairs, 16 rows of one expert possible
    (16, 320, 12, 4, 192, 5, 1, 0),           # one local expert of many
    (17, 320, 12, 3, 192, 0, 12, 1),          # 17 tokens
    (13, 320, 12, 5, 192, 0, 12, 1),          # 65 pairs
    (4, 512, 240, 8, 128, 60, 120, 1),        # two passes of two tokens
    (5, 512, 240, 8, 128, 0, 240, 1),         # ... a third would be needed
    (2, 448, 300, 8, 64, 299, 1, 0),          # two passes of one token, no or one local row
    (1, 128, 512, 64, 64, 0, 512, 1),         # 64 slots
    (2, 128, 130, 8, 64, 129, 1, 1),
])
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("load", ["even", "equal"])
def test_forward_of_few_tokens(T, d, E, k, f, eb, ec, renorm, fold, load):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T * 1000 + d + E)
    bf = lambda *s, std=1.0: torch.randn(*s, generator=gen, device=DEV).mul_(std).bfloat16()
    x, logits = bf(T, d), torch.randn(T, E, generator=gen, device=DEV)
    if load == "equal":                        # every token has the same experts, and ties among the logits
        logits[:] = (logits[:1] * 2).round()
    w = bf(ec, f, d, std=0.03), bf(ec, f, d, std=0.03), bf(ec, d, f, std=0.03)
    layer = B.MoELayerBuffers(T, d, E, k, f, eb, ec, renorm, DEV, gather=not fold, fold=fold)
    for again in range(2):                     # the second pass finds what the first one left
        layer.run_fwd(x, logits, *w)
    z = lambda *s, dt=torch.int32: torch.zeros(*s, dtype=dt, device=DEV)
    o = {"topk_idx": z(T, k), "topk_w": z(T, k, dt=torch.float32), "expert_offsets": z(ec + 1), "row_token": z(T * k), "slot_row": z(T, k)}
    o.update({n: z(T * k, c, dt=torch.bfloat16) for n, c in (("g", f), ("u", f), ("h", f), ("yp", d))}, out=z(T, d, dt=torch.bfloat16))
    ws = z(max(B.moe_workspace_bytes(T, E, k, d, f), 256), dt=torch.uint8)
    rw = z(T * k, dt=torch.float32) if fold else None
    B.moe_route_permute(logits, None, k, renorm, eb, ec, o["topk_idx"], o["topk_w"], o["expert_offsets"], o["row_token"], o["slot_row"],
                        rw, None, ws)
    guhy = [o[n] for n in ("g", "u", "h", "yp")]
    if fold:
        B.moe_grouped_gemm_fwd_folded(x, o["row_token"], rw, o["expert_offsets"], *w, *guhy)
        B.moe_unpermute_sum(o["yp"], o["slot_row"], o["out"])
    else:
        B.moe_grouped_gemm_fwd_gather(x, o["row_token"], o["expert_offsets"], *w, *guhy)
        B.moe_unpermute_combine(o["yp"], o["slot_row"], o["topk_w"], o["out"])
    rows = int(o["expert_offsets"][-1])
    assert rows == int((o["slot_row"] >= 0).sum())
    if fold:
        assert torch.equal(layer.row_weight[:rows], rw[:rows])
    for n, want in o.items():
        got = getattr(layer, n)
        if n in ("row_token", "g", "u", "h", "yp"):   # rows behind the last are nobody's
            got, want = got[:rows], want[:rows]
        assert torch.equal(got.view(want.shape), want), n
        if want.is_floating_point():
            assert bool(torch.isfinite(want).all()), n


# Buffers that share memory where the stages one by one allow it, since one of them is done with when the other is written: `a` is laid at
# the start of `b`.  1 to 4 tokens take both kernels of several stages, 16 the first, unless the memory that is shared forbids it.
@pytest.mark.parametrize("T", [1, 4, 16])
@pytest.mark.parametrize("a,b", [
    ("topk_idx", "g"), ("topk_idx", "u"), ("topk_idx", "h"), ("topk_idx", "yp"), ("topk_idx", "out"), ("topk_idx", "row_token"),
    ("topk_idx", "slot_row"), ("topk_w", "g"), ("topk_w", "h"), ("topk_w", "yp"), ("row_token", "yp"), ("row_weight", "yp"), ("row_weight", "topk_w"),
    ("row_token", "out"), ("expert_offsets", "out"), ("logits", "topk_idx"), ("logits", "h"), ("logits", "yp"), ("logits", "out"), ("x", "out"), ("x", "yp")])
@pytest.mark.parametrize("fold", [False, True])
def test_buffers_that_share_memory(T, a, b, fold):
    if not fold and (a == "topk_w" or "row_weight" in (a, b)):
        return                                  # the combine reads topk_w; there is no row_weight
    E, k, d, f = 24, 4, 320, 192
    if (a, b) == ("logits", "topk_idx"):
        E = 4                                   # as long as topk_idx
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    bf = lambda *s, std=1.0: torch.randn(*s, generator=gen, device=DEV).mul_(std).bfloat16()
    x, logits = bf(T, d), torch.randn(T, E, generator=gen, device=DEV)
    w = bf(E, f, d, std=0.05), bf(E, f, d, std=0.05), bf(E, d, f, std=0.05)
    layers = [B.MoELayerBuffers(T, d, E, k, f, 0, E, 1, DEV, gather=not fold, fold=fold) for _ in range(2)]
    layers[0].run_fwd(x, logits, *w)
    m, given = layers[1], {"x": x, "logits": logits}
    room = getattr(m, b).view(-1).view(torch.uint8)
    old = given.get(a, getattr(m, a, None))
    laid = room[:old.numel() * old.element_size()].view(old.dtype).view(old.shape)
    for again in range(2):
        if a in given:
            laid.copy_(given[a])
            m.run_fwd(*[laid if n == a else given[n] for n in ("x", "logits")], *w)
        else:
            setattr(m, a, laid)
            m.run_fwd(x, logits, *w)
        torch.cuda.synchronize()
        assert torch.equal(m.out, layers[0].out)


# Which of the two kernels a call takes, on both sides of the rules: selections in a row times workgroups for the first, one workgroup per compute
# unit and not all weights through a few of them for the second; each without the other
@pytest.mark.parametrize("T,d,E,k,f,ec,front,back", [
    (1, 2048, 64, 8, 1024, 64, True, True),
    (2, 128, 294, 32, 1920, 294, False, False),       # 64 winners in a row, 3840 workgroups
    (4, 320, 174, 16, 2048, 174, False, False),
    (1, 64, 64, 10, 128, 64, True, False), (1, 64, 64, 11, 128, 64, False, False),
    (8, 64, 64, 8, 512, 64, True, False), (8, 64, 64, 8, 576, 64, False, False), (9, 64, 8, 1, 64, 8, False, False),
    (4, 64, 240, 5, 128, 240, True, True), (4, 64, 240, 6, 128, 240, False, True),      # two passes of two tokens
    (5, 64, 240, 1, 128, 240, False, False), (2, 64, 300, 1, 128, 300, True, True), (3, 64, 300, 1, 128, 300, False, True),   # a third pass
    (4, 1024, 8, 2, 128, 8, True, True), (4, 1088, 8, 2, 128, 8, True, False), (5, 64, 8, 2, 128, 8, True, False),
    (1, 128, 64, 8, 1024, 64, True, True), (1, 128, 64, 8, 1088, 64, True, False), (1, 128, 64, 8, 1088, 32, True, True),
])
@pytest.mark.parametrize("fold", [False, True])
def test_which_kernels_a_call_takes(T, d, E, k, f, ec, front, back, fold):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T + d + E)
    bf = lambda *s, std=1.0: torch.randn(*s, generator=gen, device=DEV).mul_(std).bfloat16()
    layer = B.MoELayerBuffers(T, d, E, k, f, 0, ec, 1, DEV, gather=not fold, fold=fold)
    B.moe_prof_enable(True)
    try:
        layer.run_fwd(bf(T, d), torch.randn(T, E, generator=gen, device=DEV), bf(ec, f, d, std=0.05), bf(ec, f, d, std=0.05), bf(ec, d, f, std=0.05))
        torch.cuda.synchronize()
        names = {n for n, _, _ in B.moe_prof_read()}
    finally:
        B.moe_prof_enable(False)
    assert ("route+gate_up" in names, "down+combine" in names) == (front, back), names
    assert len(names) == 4 - front - back


# Logits at the ends of the fp32 range and NaNs through the first kernel: the routing arrays of the stage by itself, bit for bit
ENDS = [float("inf"), -float("inf"), 3.4028235e38, -3.4028235e38, 1e-45, -1e-45, 0.0, -0.0, 1.0, -1.0]


@pytest.mark.parametrize("T,E,k", [(7, 7, 7), (7, 16, 9), (7, 31, 9), (8, 64, 8), (4, 100, 9), (8, 128, 5), (2, 256, 9), (1, 512, 9)])
@pytest.mark.parametrize("nan", [False, True])
@pytest.mark.parametrize("fold", [False, True])
def test_logits_at_the_ends_of_the_range(T, E, k, nan, fold):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(E + k)
    values = torch.tensor(ENDS, device=DEV)
    if nan:
        bits = [0x7FC00000, 0xFFC00000, 0xFFFFFFFF, 0xFFFFFFFE, 0x7F800001, 0xFF800000, 0x3F800000]
        values = torch.tensor([b - (1 << 32) if b >> 31 else b for b in bits], dtype=torch.int32, device=DEV).view(torch.float32)
    logits = values.view(torch.int32)[torch.randint(0, len(values), (T, E), generator=gen, device=DEV)].view(torch.float32)
    d = f = 64
    eb, ec = (1, E - 2) if E > 7 else (0, E)
    x = torch.randn(T, d, generator=gen, device=DEV).bfloat16()
    w = [torch.randn(ec, 64, 64, generator=gen, device=DEV).mul_(0.05).bfloat16() for _ in range(3)]
    layer = B.MoELayerBuffers(T, d, E, k, f, eb, ec, 0, DEV, gather=not fold, fold=fold)
    B.moe_prof_enable(True)
    try:
        layer.run_fwd(x, logits, *w)
        torch.cuda.synchronize()
        assert "route+gate_up" in {n for n, _, _ in B.moe_prof_read()}
    finally:
        B.moe_prof_enable(False)
    z = lambda *s, dt=torch.int32: torch.zeros(*s, dtype=dt, device=DEV)
    o = {"topk_idx": z(T, k), "topk_w": z(T, k, dt=torch.float32), "expert_offsets": z(ec + 1), "row_token": z(T * k), "slot_row": z(T, k)}
    B.moe_route_permute(logits, None, k, 0, eb, ec, *[o[n] for n in o], z(T * k, dt=torch.float32) if fold else None, None, z(1 << 20, dt=torch.uint8))
    rows = int(o["expert_offsets"][-1])
    for n, want in o.items():
        got = getattr(layer, n)
        if n == "row_token":
            got, want = got[:rows], want[:rows]
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), n
    assert int(o["topk_idx"].min()) >= 0 and int(o["topk_idx"].max()) < E


# The refused backward of test_gpu_layer_buffers.py behind a forward pass of few tokens: both kernels, the first alone (8 tokens)
@pytest.mark.parametrize("name", ["dout", "dyp", "dgate", "dxp", "dWd"])
@pytest.mark.parametrize("value", [0, 4])
@pytest.mark.parametrize("path,T,E,k", [("gather", 1, 24, 4), ("gather", 8, 24, 4), ("fold", 1, 24, 4), ("fold", 8, 24, 4)])
def test_a_refused_backward_leaves_the_forward_pass_of_few_tokens(path, T, E, k, name, value):
    L.test_a_refused_backward_leaves_the_forward_pass(path, T, E, k, name, value)
