"""Selection on values at the ends of the fp32 range, for every lane group of the routing kernel, in the plain launch, the counting
one and the one of a single workgroup.  The order is that of the values, equal ones by expert id; which NaN comes first is not
defined, but no expert is chosen twice."""
import numpy as np
import pytest
import torch

from paper_2604_00785_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ENDS = np.array([np.inf, -np.inf, 3.4028235e38, -3.4028235e38, 1e-45, -1e-45, 0.0, -0.0, 1.0, -1.0], dtype=np.float32)


def _choose(logits, k, T, E):
    idx, w = torch.full((T, k), -1, dtype=torch.int32, device=DEV), torch.zeros(T, k, device=DEV)
    B.moe_route(logits, k, 0, idx, w)
    idx2, w2 = torch.full_like(idx, -1), torch.zeros_like(w)
    z = lambda *s: torch.zeros(*s, dtype=torch.int32, device=DEV)
    ws = torch.zeros(max(B.moe_permute_workspace_bytes(T, k, E), 256), dtype=torch.uint8, device=DEV)
    B.moe_route_permute(logits, None, k, 0, 0, E, idx2, w2, z(E + 1), z(T * k), z(T, k), None, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx2)
    return idx.cpu().numpy()


@pytest.mark.parametrize("E", [7, 16, 31, 64, 100, 256, 512])
@pytest.mark.parametrize("T", [3, 400])
def test_order_at_the_ends_of_the_range(E, T):
    print(f"route ends E={E} T={T}", flush=True)
    rng = np.random.default_rng(E)
    k = min(E, 9)
    v = ENDS[rng.integers(0, len(ENDS), (T, E))]
    want = np.argsort(-v.astype(np.float64), axis=1, kind="stable")[:, :k]     # stable: equal values by expert id, -0 with +0
    assert np.array_equal(_choose(torch.from_numpy(v).to(DEV), k, T, E), want)


@pytest.mark.parametrize("E,k", [(7, 7), (64, 12), (100, 20), (200, 40), (512, 70)])
def test_no_expert_is_chosen_twice_among_nans(E, k):
    print(f"route nan E={E} k={k}", flush=True)
    rng = np.random.default_rng(E + k)
    T = 5
    bits = rng.choice(np.array([0x7FC00000, 0xFFC00000, 0xFFFFFFFF, 0xFFFFFFFE, 0x7F800001, 0xFF800000, 0x3F800000], dtype=np.uint32), (T, E))
    bits[0] = 0xFFFFFFFF
    idx = _choose(torch.from_numpy(bits.view(np.float32)).to(DEV), k, T, E)
    assert idx.min() >= 0 and idx.max() < E
    assert all(len(set(r)) == k for r in idx.tolist())
