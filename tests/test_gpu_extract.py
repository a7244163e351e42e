"""The tile form of the greedy extraction (large exact shapes) against the
per-occupancy kernel, which a batch of one instance takes: the same policy
bytes and gap bits, at each tile depth, with ragged last chunks, the smallest
shapes the form takes and ones just below, ties, infinities and NaN."""
import pytest

import workloads as W
from tests.gpu_util import torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mdpvi():
    torch_cuda()
    import paper_2012_12419_amd as m
    m.load()
    return m


# (K, C, sizes): tile depths 2, 3 and 4; tiles of a multiple of 4 occupancies,
# of odd and of 2 mod 4; the fewest tiles and occupancies (256 of each)
@pytest.mark.parametrize("K,C,size", [(4, 15, [1, 2, 3]), (4, 16, [3]), (4, 14, [1, 2]), (5, 15, [2, 1]), (6, 7, [1, 2, 4]),
                                      (6, 10, [1, 2, 4]), (6, 9, [1, 9]), (7, 6, [1, 2, 3]), (7, 6, [6]),
                                      (8, 3, [1, 2, 3]), (8, 3, [1]), (8, 4, [4, 1])])
def test_tiles_equal_single_occupancies(mdpvi, K, C, size):
    import torch
    J = len(size)
    p = W.make(K, C, size, [0.7 / (1 + j) for j in range(J)], 0.1, 0.02, [1.1 * (1 + j) for j in range(J)], 0.9,
               reject_cost=[0.2 + 0.1 * j for j in range(J)], idle_unit_cost=0.03)
    mdp, batch = mdpvi.MDP.from_instance(p), mdpvi.Batch([p])
    g = torch.Generator(device="cuda").manual_seed(K * 31 + C)
    noise = torch.randn(p.num_states, generator=g, device="cuda", dtype=torch.float64)
    special = noise.clone()
    pick = torch.randint(0, p.num_states, (2000,), generator=g, device="cuda")
    special[pick[:700]] = float("inf")
    special[pick[700:1400]] = -float("inf")
    special[pick[1400:]] = float("nan")
    for dtype, bits in ((torch.float32, torch.int32), (torch.float64, torch.int32)):
        for V in (noise, (noise * 2).round(), special):
            V = V.to(dtype)
            pi, gap = mdp.policy_extract(V)
            ref, rgap = batch.policy_extract(V)
            assert torch.equal(pi, ref)
            num = ~torch.isnan(rgap)
            assert torch.equal(torch.isnan(gap), ~num) and torch.equal(gap[num].view(bits), rgap[num].view(bits))
            assert torch.equal(mdp.policy_extract(V, want_gap=False)[0], ref)
