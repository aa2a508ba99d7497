"""A row's results are a function of its token and its expert's weights, bit for bit: not of the expert's number, of the share of the experts that
a call holds, nor of the kernel that takes the row.  Reductions of 32 steps and more, weight rows of one, two and three times 4096 bytes."""
import pytest
import torch

import gpu_harness as H
from paper_2604_00785_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _normal(gen, *s, std=1.0):
    return torch.randn(*s, generator=gen, device=DEV).mul_(std).bfloat16()


# every expert has the same weights and the same rows; edge 0: the rule's kernels (streaming up to 8 rows per expert)
@pytest.mark.parametrize("d,f", [(2048, 128), (128, 2048), (4096, 64), (64, 6144), (1088, 192)])
@pytest.mark.parametrize("rows,edge", [(3, 0), (3, 128), (70, 128), (70, 256), (300, 256)])
def test_no_result_depends_on_the_number_of_the_expert(d, f, rows, edge, monkeypatch):
    E = 33
    gen = torch.Generator(device=DEV)
    gen.manual_seed(d + f + rows)
    one = _normal(gen, f, d, std=0.05), _normal(gen, f, d, std=0.05), _normal(gen, d, f, std=0.05)
    w = [t.expand(E, -1, -1).contiguous() for t in one]
    xp = _normal(gen, rows, d).repeat(E, 1)
    off = torch.arange(E + 1, device=DEV, dtype=torch.int32) * rows
    out = [torch.full((E * rows, n), float("nan"), dtype=torch.bfloat16, device=DEV) for n in (f, f, f, d)]
    if edge:
        lib = H.AtEdge(edge)
        monkeypatch.setattr(B, "load", lambda: lib)
    B.moe_grouped_gemm_fwd(xp, off, *w, *out)
    torch.cuda.synchronize()
    for n, t in zip(("g", "u", "h", "yp"), out):
        t = t.view(E, rows, -1)
        assert bool(torch.isfinite(t).all()), n
        assert torch.equal(t, t[:1].expand_as(t)), n


# the rows of a share of the experts against those of the whole layer, in calls that take one kernel for several stages (1, 4, 8 tokens),
# streaming products (1, 24) and tiled ones
@pytest.mark.parametrize("T,d,f", [(1, 2048, 2048), (4, 2048, 128), (8, 4096, 64), (24, 2048, 2048), (300, 2048, 64), (300, 64, 2048)])
@pytest.mark.parametrize("path", ["plain", "gather", "fold"])
def test_a_share_of_the_experts_has_the_rows_of_the_whole_layer(T, d, f, path):
    E, k, eb, ec = 12, 6, 3, 7
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T + d + f)
    x, logits = _normal(gen, T, d), torch.randn(T, E, generator=gen, device=DEV)
    w = _normal(gen, E, f, d, std=0.03), _normal(gen, E, f, d, std=0.03), _normal(gen, E, d, f, std=0.03)
    layer = lambda b, n: B.MoELayerBuffers(T, d, E, k, f, b, n, 1, DEV, gather=path == "gather", fold=path == "fold")
    whole, share = layer(0, E), layer(eb, ec)
    whole.run_fwd(x, logits, *w)
    share.run_fwd(x, logits, *[t[eb:eb + ec].contiguous() for t in w])
    torch.cuda.synchronize()
    assert torch.equal(whole.topk_idx, share.topk_idx) and torch.equal(whole.topk_w, share.topk_w)
    first = int(whole.expert_offsets[eb])
    assert torch.equal(whole.expert_offsets[eb:eb + ec + 1] - first, share.expert_offsets)
    rows = int(share.expert_offsets[-1])
    assert rows > 0
    for n in ("row_token", "g", "u", "h", "yp"):
        assert torch.equal(getattr(whole, n)[first:first + rows], getattr(share, n)[:rows]), n
