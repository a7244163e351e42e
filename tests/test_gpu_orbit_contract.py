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


# A chosen form evaluates by full sweeps: the bits of the form with orbits off.
# first and last: the forms of one instance with and without orbit LDS solves.
@pytest.mark.parametrize("K,C,J", [(3, 8, 2), (5, 10, 2)])
def test_chosen_sweep_forms_are_run(mdpvi, K, C, J):
    import torch
    p = _inst(K, C, J)
    pi = mdpvi.MDP.from_instance(p).policy_greedy("least_loaded")
    forms = [0, -1] + ([mdpvi.FORM_TILE] if K >= 4 else [])

    def run(form=None, orbits=None):
        mdp = mdpvi.MDP.from_instance(p)
        if orbits is not None:
            mdp.set_orbits(orbits)
        if form is not None:
            mdp.set_sweep_form(form)
        V, _ = mdp.policy_eval(pi, tol=1e-10)
        q = pi.clone()
        V2 = torch.zeros_like(V)
        mdp.policy_iteration(q, V2, eval_tol=1e-10, improve_tol=1e-8, max_rounds=20)
        return V, V2

    full = run(0, False)
    free = run()
    assert not torch.equal(free[0], full[0])   # the orbit sums round otherwise at these shapes
    for f in forms:
        for x, y in zip(run(f), full):
            assert torch.equal(x, y), f
        for x, y in zip(run(f, True), free):   # asked for by name: on in every form
            assert torch.equal(x, y), f


def test_chosen_batch_forms_are_run(mdpvi):
    import torch
    insts = [_inst(3, 8, 2), _inst(5, 10, 2), _inst(4, 12, 3)]

    def run(choose=lambda b: None):
        b = mdpvi.Batch(insts)
        choose(b)
        pi = b.policy_greedy("least_loaded")
        V = b.policy_eval(pi, tol=1e-10)[0]
        V2 = torch.zeros_like(V)
        b.policy_iteration(pi, V2, eval_tol=1e-10, improve_tol=1e-8)
        return V, V2

    full = run(lambda b: b.set_orbits(False))
    free = run()
    assert not torch.equal(free[0], full[0])
    for choose in (lambda b: b.set_round_form("eval", 2), lambda b: b.set_round_form("eval", 0),
                   lambda b: b.set_tile_form("eval", 1), lambda b: b.set_tile_form("eval", 0)):
        for x, y in zip(run(choose), full):
            assert torch.equal(x, y)

        def both(b):
            b.set_orbits(True)
            choose(b)
        for x, y in zip(run(both), free):
            assert torch.equal(x, y)
    for op in ("vi", "adjoint"):   # of another operation: nothing to the evaluation
        for x, y in zip(run(lambda b: b.set_round_form(op, 2)), free):
            assert torch.equal(x, y)


# More units than the exact sums' 2^21 range of values has room for (K C > 256):
# 300, 540 and 264 of them, launched sweeps with 16- and 32-bit tables.
@pytest.mark.parametrize("K,C", [(3, 100), (3, 180), (4, 66)])
def test_same_bits_over_the_stated_range(mdpvi, K, C):
    """Value iteration from an invariant start whose values spread over the
    factor 2^29 / (K C) that the header states: the full sweeps' bits."""
    import math
    import torch
    p = _inst(K, C, 1, gamma=0.95)
    g = torch.Generator(device="cuda").manual_seed(K * C)
    per_digit = torch.rand(C + 1, generator=g, device="cuda", dtype=torch.float64)
    o = torch.arange(p.num_states, device="cuda")
    u = torch.zeros(p.num_states, dtype=torch.float64, device="cuda")
    digits = torch.stack([o // (C + 1) ** k % (C + 1) for k in range(K)]).sort(dim=0).values
    for d in digits:                       # in the order of the sorted digits: the same bits over an orbit
        u = (u + 7 * per_digit[d]) % 1.0
    V0 = torch.exp2(u * math.log2(2 ** 29 / (K * C))).float()
    outs = []
    for orbits in (True, False):
        mdp = mdpvi.MDP.from_instance(p)
        mdp.set_orbits(orbits)
        V = V0.clone()
        with pytest.raises(mdpvi.MdpviError) as e:
            mdp.vi_solve(V, tol=1e-30, max_iter=40)
        assert e.value.code == mdpvi.ENOCONV
        outs.append((V, e.value.stats["residual_inf"]))
    assert outs[0][1] == outs[1][1] and torch.equal(outs[0][0].view(torch.int32), outs[1][0].view(torch.int32))
