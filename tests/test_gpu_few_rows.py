"""GPU parity of the variants that calls with few rows take, at the sizes where a tile, a lane group or a wave's share
ends.  Same oracle, inputs and tolerances as the tests they reuse."""
import numpy as np
import pytest
import torch

import gpu_harness as H
import test_gpu_parity as P
from paper_2604_00785_amd import binding as B

pytestmark = pytest.mark.gpu


# few rows per expert, on both sides of the rule of the products that stream the weights (at most 8 rows per expert on average
# where the calls know no number of tokens)
@pytest.mark.parametrize("counts,d,f", [
    ([1] * 8 + [0, 0], 64, 64),
    ([16, 0, 17, 0, 1, 33, 0, 0, 15, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0], 192, 128),     # rows at and past 16
    ([2, 0, 9] * 40 + [0] * 10, 320, 192),            # more than 64 experts
    ([32, 33, 0, 31, 1, 64, 3, 2, 7, 0, 0, 0], 448, 320),
    ([20] * 130, 128, 64),                            # more than 128 experts
])
def test_streamed_products(counts, d, f):
    P.test_grouped_gemm_fwd_bwd_isolated(counts, d, f)


# the streamed products themselves (R_cap = rows + 37 is at most 8 per expert)
@pytest.mark.parametrize("counts,d,f", [
    ([1] * 8 + [0] * 4, 64, 64),                              # one piece of the reduction
    ([16, 0, 17, 0, 1, 33, 0, 0, 15] + [0] * 22, 192, 128),   # rows at and past a 16-row tile; three pieces
    ([2, 0, 9] * 40 + [0] * 10, 320, 192),                    # more than 64 experts; five pieces
    ([3] * 130, 128, 64),                                     # more than 128 experts
    ([5, 0, 1, 18] + [0] * 12, 2048, 1088),                   # 32 and 17 pieces, two waves per tile
    ([4, 2, 1] * 8 + [0] * 12, 1088, 2048),                   # 17 and 32 pieces, one wave per tile in gate/up
])
def test_streamed_products_alone(counts, d, f):
    assert sum(counts) + 37 <= 8 * len(counts)
    P.test_grouped_gemm_fwd_bwd_isolated(counts, d, f)


# whole layers whose experts have few rows, in each form, with wide and uneven reductions
@pytest.mark.parametrize("T,d,E,k,f,eb,ec,renorm", [
    (1, 2048, 16, 8, 1024, 0, 16, 1),     # a decoding step of one sequence
    (31, 1088, 24, 4, 576, 0, 24, 0),     # 17 and 9 pieces
    (48, 576, 40, 3, 1088, 0, 40, 1),     # more than 32 tokens, at most 8 rows per expert
    (17, 2048, 30, 6, 192, 11, 7, 0),     # a rank's share, 17 rows of one expert possible
    (70, 1088, 64, 4, 192, 8, 4, 1),      # a rank's share, few rows expected: decided on the device
    (2, 1088, 16, 2, 448, 0, 16, 1),      # blocks of two pieces, the last one half: 17 and 7 pieces
])
@pytest.mark.parametrize("form", ["plain", "gather", "fold"])
def test_layer_with_few_rows(T, d, E, k, f, eb, ec, renorm, form):
    {"plain": P.test_layer_ragged_shapes, "gather": P.test_layer_gathered_rows, "fold": P.test_layer_folded_gate_weights}[form](
        T, d, E, k, f, eb, ec, renorm)


# The streamed products give the bits of the tiled ones: the same rows through a call whose capacity or number of tokens
# is too large for them.
@pytest.mark.parametrize("T,d,E,k,f", [(1, 2048, 16, 8, 1024), (9, 1088, 40, 8, 576), (32, 512, 24, 20, 2048), (40, 2048, 150, 9, 192), (20, 64, 5, 5, 64), (3, 1088, 16, 2, 448)])
@pytest.mark.parametrize("form", ["plain", "gather", "fold"])
def test_streamed_products_have_the_bits_of_the_tiled(T, d, E, k, f, form):
    gen = torch.Generator(device=P.DEV)
    gen.manual_seed(T + d + E)
    bf = lambda *s, std=1.0: torch.randn(*s, generator=gen, device=P.DEV).mul_(std).bfloat16()
    z = lambda *s, dt=torch.int32: torch.zeros(*s, dtype=dt, device=P.DEV)
    R, cap, tokens = T * k, T * k + 20 * E, T + 64
    x = bf(tokens, d)
    w = bf(E, f, d, std=0.03), bf(E, f, d, std=0.03), bf(E, d, f, std=0.03)
    topk_idx, topk_w, slot_row, off = z(T, k), z(T, k, dt=torch.float32), z(T, k), z(E + 1)
    row_token, row_weight, xp = z(cap), z(cap, dt=torch.float32), z(cap, d, dt=torch.bfloat16)
    ws = z(max(B.moe_workspace_bytes(T, E, k, d, f), 256), dt=torch.uint8)
    B.moe_route_permute(torch.randn(T, E, generator=gen, device=P.DEV), x[:T], k, 1, 0, E, topk_idx, topk_w, off, row_token[:R],
                        slot_row, row_weight[:R], xp[:R], ws)

    def products(c, t):
        o = [torch.full((c, n), float("nan"), dtype=torch.bfloat16, device=P.DEV) for n in (f, f, f, d)]
        if form == "plain":
            B.moe_grouped_gemm_fwd(xp[:c], off, *w, *o)
        elif form == "gather":
            B.moe_grouped_gemm_fwd_gather(x[:t], row_token[:c], off, *w, *o)
        else:
            B.moe_grouped_gemm_fwd_folded(x[:t], row_token[:c], row_weight[:c], off, *w, *o)
        assert all(bool(torch.isnan(v[R:]).all()) for v in o)
        return [v[:R].view(torch.int16) for v in o]

    tiled = products(cap, tokens)
    few = products(R, T)
    if form == "plain" and R > 8 * E:
        pytest.skip("a call that knows no number of tokens takes the tiled products")
    for n, a, b in zip("guhy", few, tiled):
        assert torch.equal(a, b), n


# A list of many tiles whose experts' sizes are in no order: several rounds of runs taken from both ends, and (more than 128
# experts) in index order, at either tile edge
@pytest.mark.parametrize("E,d,f", [(96, 1024, 1024), (72, 512, 2048), (140, 1024, 512)])
@pytest.mark.parametrize("edge", [128, 256])
def test_many_rounds_of_uneven_experts(E, d, f, edge, monkeypatch):
    rng = np.random.default_rng(E)
    counts = np.concatenate([[1100, 520, 513, 300, 257, 256, 255, 0, 0, 0], rng.integers(1, 30, E - 10)])
    rng.shuffle(counts)
    row_tiles = sum(-(-c // edge) for c in counts)
    workgroups = 256 * 256 // edge
    assert 2 * workgroups < row_tiles * (f // (edge // 2)) and row_tiles <= 3 * E      # of gate/up: more than two rounds, both ends
    lib = H.AtEdge(edge)
    monkeypatch.setattr(B, "load", lambda: lib)
    P.test_grouped_gemm_fwd_bwd_isolated([int(c) for c in counts], d, f)


# Stages 1-3 in one workgroup: at most 1024 pairs, two passes of the workgroup's 128 (up to 64 experts), 64 (128), 32 (256) or 16
# lane groups; the odd sizes here take the first call of the two launches
@pytest.mark.parametrize("T,E,k,eb,ec", [
    (128, 12, 4, 0, 12), (129, 12, 4, 2, 9), (256, 24, 4, 0, 24), (257, 24, 3, 0, 24), (64, 100, 8, 0, 100), (65, 100, 8, 7, 90),
    (128, 100, 8, 0, 100), (129, 100, 7, 0, 100), (32, 200, 9, 0, 200), (33, 200, 9, 150, 50), (64, 200, 16, 0, 200), (65, 200, 15, 0, 200)])
@pytest.mark.parametrize("renorm,gate", [(0, False), (1, True)])
def test_one_launch_routing_passes(T, E, k, eb, ec, renorm, gate):
    P.test_route_permute_one_call(T, E, k, eb, ec, renorm, gate)


# both sides of the rule for one workgroup: at most 1024 pairs and two passes
@pytest.mark.parametrize("T,E,k,eb,ec", [
    (128, 64, 8, 0, 64), (129, 64, 8, 3, 50),         # the last call of one launch, the first of two
    (65, 8, 1, 0, 8), (256, 33, 4, 1, 31), (257, 33, 3, 0, 33), (100, 130, 10, 0, 130), (14, 512, 70, 0, 512), (17, 300, 3, 299, 1)])
@pytest.mark.parametrize("renorm,gate", [(0, False), (1, True)])
def test_one_launch_routing(T, E, k, eb, ec, renorm, gate):
    P.test_route_permute_one_call(T, E, k, eb, ec, renorm, gate)


# Both variants of the streaming products on either side of their rule (384 expected tiles; weight rows of a multiple of 4096 bytes), in
# reductions of 1, 2, 3 and more steps than a ring has pieces: the bits of the tiled kernel
@pytest.mark.parametrize("d,f", [(2048, 1024), (1984, 1024), (2112, 960), (64, 1024), (128, 1024), (192, 1024), (2048, 64), (2048, 128), (2048, 192),
                                 (4096, 2048)])
@pytest.mark.parametrize("form", ["gather", "fold"])
def test_variants_of_the_streamed_products(d, f, form):
    T, E, k = 24, 24, 1
    rows = T * k
    tiles = rows * E // (rows + E)
    assert min(abs(tiles * (f // 32) - 384), abs(tiles * (d // 64) - 384)) <= 24 or (d, f) == (4096, 2048)
    test_streamed_products_have_the_bits_of_the_tiled(T, d, E, k, f, form)
