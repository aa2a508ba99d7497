"""The two tile sizes of the grouped products give the same bits: the same rows through calls of two capacities, a tight one, for
which the rule takes tiles of 128, and one so large that it expects long lists and takes tiles of 256.  (The tests against the
oracle run the sizes here and smaller ones through tiles of 128, the full-size ones through tiles of 256.)"""
import pytest
import torch

from paper_2604_00785_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# rows at and past the ends of 32-row groups, of waves and of tiles of either size; 1 to 9 reduction steps in every product; columns
# that are no multiple of 128 or 256; experts in both halves of a wave's table, and more than fit it
@pytest.mark.parametrize("counts,d,f", [
    ([1, 0, 31, 32, 33, 63, 64, 65, 96, 97], 256, 256),
    ([127, 128, 129, 0, 160, 161, 255, 256, 257], 576, 320),
    ([383, 384, 385, 1], 320, 576),
    ([511, 0, 513, 40], 448, 448),
    ([5, 130, 0, 260] * 17, 256, 320),          # 68 experts
    ([3, 129] * 66, 320, 256),                  # 132 experts: looked up per tile
])
@pytest.mark.parametrize("form", ["plain", "gather", "fold"])
def test_tile_sizes_give_the_same_bits(counts, d, f, form):
    print(f"tile sizes {form} counts={counts[:10]} d={d} f={f}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(sum(counts) + d)
    bf = lambda *s, std=1.0: torch.randn(*s, generator=gen, device=DEV).mul_(std).bfloat16()
    E, R, T = len(counts), sum(counts), 700
    off = torch.tensor([0] + counts, device=DEV).cumsum(0).to(torch.int32)
    w = bf(E, f, d, std=0.05), bf(E, f, d, std=0.05), bf(E, d, f, std=0.05)
    x, dout = bf(T, d), bf(T, d)
    big = 200000
    row_token = torch.randint(0, T, (big,), generator=gen, device=DEV, dtype=torch.int32)
    row_weight = torch.rand(big, generator=gen, device=DEV)
    slot_row = torch.full((T, 1), -1, dtype=torch.int32, device=DEV)
    slot_row[:min(R, T), 0] = torch.arange(min(R, T), device=DEV, dtype=torch.int32)
    xp, dyp = (t.index_select(0, row_token.long()) for t in (x, dout))

    def products(cap):
        nan = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device=DEV)
        g, u, h, yp, dxp = nan(cap, f), nan(cap, f), nan(cap, f), nan(cap, d), nan(cap, d)
        dW = nan(E, f, d), nan(E, f, d), nan(E, d, f)
        dgate = torch.full((T, 1), float("nan"), device=DEV)
        nbytes = B.moe_grouped_gemm_bwd_folded_workspace_bytes(cap, f) if form == "fold" else B.moe_grouped_gemm_bwd_workspace_bytes(cap, f)
        ws = torch.zeros(nbytes, dtype=torch.uint8, device=DEV)
        if form == "plain":
            B.moe_grouped_gemm_fwd(xp[:cap], off, *w, g, u, h, yp)
            B.moe_grouped_gemm_bwd(dyp[:cap], xp[:cap], g, u, h, off, *w, dxp, *dW, ws)
        elif form == "gather":
            B.moe_grouped_gemm_fwd_gather(x, row_token[:cap], off, *w, g, u, h, yp)
            B.moe_grouped_gemm_bwd_gather(dyp[:cap], x, row_token[:cap], g, u, h, off, *w, dxp, *dW, ws)
        else:
            B.moe_grouped_gemm_fwd_folded(x, row_token[:cap], row_weight[:cap], off, *w, g, u, h, yp)
            B.moe_grouped_gemm_bwd_folded(dout, x, row_token[:cap], row_weight[:cap], slot_row, g, u, h, off, *w, dxp, *dW, dgate, ws)
        torch.cuda.synchronize()
        for t in (g, u, h, yp, dxp):
            assert bool(torch.isnan(t[R:]).all())               # rows past the last expert's end are not written
            assert bool(torch.isfinite(t[:R]).all())
        for e, n in enumerate(counts):
            assert n > 0 or all(bool((t[e] == 0).all()) for t in dW)
        return [t[:R] for t in (g, u, h, yp, dxp)] + list(dW) + ([dgate] if form == "fold" else [])

    names = ["g", "u", "h", "yp", "dxp", "dWg", "dWu", "dWd", "dgate"]
    for n, a, b in zip(names, products(R + 11 * E), products(big)):
        assert torch.equal(a.view(torch.int32 if n == "dgate" else torch.int16), b.view(torch.int32 if n == "dgate" else torch.int16)), n
