"""What the orbit form of an evaluation must leave as it is: the start that a
call is given, whatever its tolerance, and the form that a caller chose."""
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


def _inst(K, C, J, gamma=0.9):
    size = [1 + j % C for j in range(J)]
    return W.make(K, C, size, [0.7 / (1 + j) for j in range(J)], 0.1, 0.02, [1.1 * (1 + j) for j in range(J)], gamma)


def _spread(V, amount):
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    return V + amount * torch.rand(V.shape, generator=g, dtype=V.dtype, device="cuda")


# solved in one workgroup's LDS, and by launched sweeps
@pytest.mark.parametrize("K,C,J", [(3, 8, 2), (5, 9, 2)])
@pytest.mark.parametrize("tol", [0.1, 1e-3, 1e300])
def test_evaluation_keeps_its_start(mdpvi, K, C, J, tol):
    """The iterates are those of the given V^0, however loose the tolerance: a
    start whose values differ within an orbit by less than tol/2 gives the
    bits of the full sweeps."""
    import torch
    p = _inst(K, C, J)
    pi = mdpvi.MDP.from_instance(p).policy_greedy("least_loaded")
    base = torch.full((p.num_states,), 3.0, dtype=torch.float64, device="cuda")
    outs = []
    for orbits in (True, False):
        mdp = mdpvi.MDP.from_instance(p)
        mdp.set_orbits(orbits)
        V = _spread(base, 0.4 * min(tol, 1.0))
        _, st = mdp.policy_eval(pi, V, tol=tol)
        outs.append((V, st["iterations"], st["residual_inf"]))
    assert outs[0][1:] == outs[1][1:] and torch.equal(outs[0][0], outs[1][0])


def test_batch_evaluation_keeps_its_start(mdpvi):
    import torch
    insts = [_inst(3, 8, 2), _inst(5, 9, 2), _inst(4, 6, 3)]
    outs = []
    for orbits in (True, False):
        b = mdpvi.Batch(insts)
        b.set_orbits(orbits)
        V = _spread(torch.full((b.num_states,), 3.0, dtype=torch.float64, device="cuda"), 0.04)
        V, _, its, res = b.policy_eval(b.policy_greedy("least_loaded"), V, tol=0.1)
        outs.append((V, its, res))
    assert outs[0][1:] == outs[1][1:] and torch.equal(outs[0][0], outs[1][0])
