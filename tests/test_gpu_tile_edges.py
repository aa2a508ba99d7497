"""The grouped products at both of their tile edges, whatever the rule would take: against the oracle, and the same bits from both.
The edge is handed to the call and the one that a launch ran with comes back (gpu_harness.AtEdge)."""
import ctypes

import pytest
import torch

import gpu_harness as H
import test_gpu_parity as P
from paper_2604_00785_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(params=[128, 256])
def at_edge(request, monkeypatch):
    lib = H.AtEdge(request.param)
    monkeypatch.setattr(B, "load", lambda: lib)
    yield request.param
    assert lib.launches >= 4                    # forward and backward, two launches each


# one, two, three and more reduction steps forward (d, f / 64) and in the weight gradients (rows / 64, whole and partial last steps),
# strips and columns past the last whole tile of either edge, rows at and past the ends of tiles, empty experts, more than fit a
# wave's table
@pytest.mark.parametrize("counts,d,f", [
    ([64, 64, 64, 64], 128, 256), ([300, 0, 5, 257, 256, 1, 0, 700], 192, 320), ([1100, 900], 512, 128), ([0, 0, 40], 64, 64),
    ([70, 1, 63, 64, 65, 128, 320, 330, 449], 64, 64), ([130, 130, 130], 320, 448), ([257, 511], 384, 704), ([3] * 130, 64, 128),
    ([300 if e % 9 == 0 else 7 for e in range(100)], 64, 128),
    ([257, 40, 129, 0, 191], 64, 192), ([96, 511, 1, 33], 128, 64), ([255, 160, 513], 192, 128), ([31, 400, 97], 128, 128),
])
def test_products_against_the_oracle(at_edge, counts, d, f):
    P.test_grouped_gemm_fwd_bwd_isolated(counts, d, f)


@pytest.mark.parametrize("seed", range(8))
def test_random_products_against_the_oracle(at_edge, seed):
    P.test_grouped_gemm_random_shapes(seed)


# the rule itself, on calls whose experts have no rows: a small layer and a large one
@pytest.mark.parametrize("E,R_cap,d,f,edge", [(8, 512, 128, 256, 128), (64, 65536, 2048, 1024, 256)])
def test_rule_takes_either_edge(E, R_cap, d, f, edge):
    lib = H.AtEdge(0).lib
    z = lambda *s, dt=torch.bfloat16: torch.zeros(*s, dtype=dt, device=DEV)
    off, buf, weights, ws = z(E + 1, dt=torch.int32), z(8, max(d, f)), z(E * d * f), z(256, dt=torch.uint8)
    dw = [z(E * d * f) for _ in range(3)]
    rows, w = buf.data_ptr(), [weights.data_ptr()] * 3                    # no row is read or written
    nbytes = B.moe_grouped_gemm_bwd_workspace_bytes(R_cap, f)             # only rows of it would be written
    fwd, bwd = (ctypes.c_int * 2)(), (ctypes.c_int * 2)()
    assert lib.moe_gemm_fwd(rows, None, None, off.data_ptr(), *w, E, R_cap, R_cap, R_cap, d, f, rows, rows, rows, rows, B._stream(),
                            ctypes.addressof(fwd)) == 0
    assert lib.moe_gemm_bwd(rows, rows, 0, None, rows, rows, rows, off.data_ptr(), *w, E, R_cap, R_cap, d, f, rows,
                            *[t.data_ptr() for t in dw], ws.data_ptr(), nbytes, B._stream(), ctypes.addressof(bwd)) == 0
    torch.cuda.synchronize()
    assert list(fwd) + list(bwd) == [edge] * 4


# rows at and past the ends of 32-row groups, of waves and of tiles of either size; 1 to 9 reduction steps in every product; columns
# that are no multiple of 128 or 256; experts in both halves of a wave's table, and more than fit it
@pytest.mark.parametrize("counts,d,f", [
    ([70, 1, 63, 64, 65, 128, 320, 330, 449], 64, 64),
    ([257, 40, 129, 0, 191], 64, 192),
    ([96, 511, 1, 33], 192, 128),
    ([1, 0, 31, 32, 33, 63, 64, 65, 96, 97], 256, 256),
    ([127, 128, 129, 0, 160, 161, 255, 256, 257], 576, 320),
    ([383, 384, 385, 1], 320, 576),
    ([511, 0, 513, 40], 448, 448),
    ([5, 130, 0, 260] * 17, 256, 320),          # 68 experts
    ([3, 129] * 66, 320, 256),                  # 132 experts: looked up per tile
])
@pytest.mark.parametrize("form", ["plain", "gather", "fold"])
def test_tile_sizes_give_the_same_bits(counts, d, f, form, monkeypatch):
    print(f"tile sizes {form} counts={counts[:10]} d={d} f={f}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(sum(counts) + d)
    bf = lambda *s, std=1.0: torch.randn(*s, generator=gen, device=DEV).mul_(std).bfloat16()
    E, R, T = len(counts), sum(counts), 700
    off = torch.tensor([0] + counts, device=DEV).cumsum(0).to(torch.int32)
    w = bf(E, f, d, std=0.05), bf(E, f, d, std=0.05), bf(E, d, f, std=0.05)
    x, dout = bf(T, d), bf(T, d)
    cap = R + 37
    row_token = torch.randint(0, T, (cap,), generator=gen, device=DEV, dtype=torch.int32)
    row_weight = torch.rand(cap, generator=gen, device=DEV)
    slot_row = torch.full((T, 1), -1, dtype=torch.int32, device=DEV)
    slot_row[:min(R, T), 0] = torch.arange(min(R, T), device=DEV, dtype=torch.int32)
    xp, dyp = (t.index_select(0, row_token.long()) for t in (x, dout))

    def products(edge, form):
        lib = H.AtEdge(edge)
        monkeypatch.setattr(B, "load", lambda: lib)
        nan = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device=DEV)
        g, u, h, yp, dxp = nan(cap, f), nan(cap, f), nan(cap, f), nan(cap, d), nan(cap, d)
        dW = nan(E, f, d), nan(E, f, d), nan(E, d, f)
        dgate = torch.full((T, 1), float("nan"), device=DEV)
        nbytes = B.moe_grouped_gemm_bwd_folded_workspace_bytes(cap, f) if form == "fold" else B.moe_grouped_gemm_bwd_workspace_bytes(cap, f)
        ws = torch.zeros(nbytes, dtype=torch.uint8, device=DEV)
        if form == "plain":
            B.moe_grouped_gemm_fwd(xp, off, *w, g, u, h, yp)
            B.moe_grouped_gemm_bwd(dyp, xp, g, u, h, off, *w, dxp, *dW, ws)
        elif form == "gather":
            B.moe_grouped_gemm_fwd_gather(x, row_token, off, *w, g, u, h, yp)
            B.moe_grouped_gemm_bwd_gather(dyp, x, row_token, g, u, h, off, *w, dxp, *dW, ws)
        else:
            B.moe_grouped_gemm_fwd_folded(x, row_token, row_weight, off, *w, g, u, h, yp)
            B.moe_grouped_gemm_bwd_folded(dout, x, row_token, row_weight, slot_row, g, u, h, off, *w, dxp, *dW, dgate, ws)
        torch.cuda.synchronize()
        for t in (g, u, h, yp, dxp):
            assert bool(torch.isnan(t[R:]).all())               # rows past the last expert's end are not written
            assert bool(torch.isfinite(t[:R]).all())
        for e, n in enumerate(counts):
            assert n > 0 or all(bool((t[e] == 0).all()) for t in dW)
        monkeypatch.undo()
        return [t[:R] for t in (g, u, h, yp, dxp)] + list(dW) + ([dgate] if form == "fold" else [])

    names = ["g", "u", "h", "yp", "dxp", "dWg", "dWu", "dWd", "dgate"]
    small, large = products(128, form), products(256, form)
    others = [small] + ([products(256, "plain")] if form == "gather" else [])     # the same rows, materialised
    for other in others:
        for n, a, b in zip(names, other, large):
            assert torch.equal(a.view(torch.int32 if n == "dgate" else torch.int16), b.view(torch.int32 if n == "dgate" else torch.int16)), n


# Reductions of 32 and 64 steps and of weight rows that are multiples of 4096 bytes, beside tiles that hold all rows of an expert
@pytest.mark.parametrize("counts,d,f", [([70, 1, 0, 130, 300], 2048, 64), ([65, 3, 257], 64, 2048), ([40, 129], 4096, 128)])
@pytest.mark.parametrize("form", ["plain", "gather", "fold"])
def test_tile_sizes_give_the_same_bits_in_long_reductions(counts, d, f, form, monkeypatch):
    test_tile_sizes_give_the_same_bits(counts, d, f, form, monkeypatch)
