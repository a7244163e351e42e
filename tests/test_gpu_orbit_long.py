"""Solves in one workgroup's LDS at their limits: more sweeps than one launch
holds (8,192), so that iterates and arrival terms go through device memory
between launches, alone and in a batch beside an instance that stops early and
one that the form refuses; and the shapes with the most LDS (157,336 bytes of
value iteration at K = 2, C = 113, 149,008 of evaluation at K = 2, C = 95)."""
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


def _inst(K, C, J, gamma):
    size = [1 + j % C for j in range(J)]
    return W.make(K, C, size, [0.7 / (1 + j) for j in range(J)], 0.1, 0.02, [1.1 * (1 + j) for j in range(J)], gamma)


def _rounding(p):
    # as derived in test_gpu_orbit.py: 4 K + 8 roundings a sweep differ, contracted by gamma
    return 2 * (4 * p.K + 8) * 2.0 ** -53 / (1 - p.gamma)


def _vi(mdpvi, p, orbits, V0, tol, most):
    mdp = mdpvi.MDP.from_instance(p)
    mdp.set_orbits(orbits)
    V = V0.clone()
    try:
        st = mdp.vi_solve(V, tol=tol, max_iter=most)
    except mdpvi.MdpviError as e:
        assert e.code == mdpvi.ENOCONV
        st = e.stats
    return V, st["iterations"], st["residual_inf"]


def _ev(mdpvi, p, orbits, tol, most):
    mdp = mdpvi.MDP.from_instance(p)
    mdp.set_orbits(orbits)
    import torch
    V = torch.zeros(p.num_states, dtype=torch.float64, device="cuda")
    try:
        st = mdp.policy_eval(mdp.policy_greedy("least_loaded"), V, tol=tol, max_iter=most)[1]
    except mdpvi.MdpviError as e:
        assert e.code == mdpvi.ENOCONV
        st = e.stats
    return V, st["iterations"], st["residual_inf"]


# to the FP32 fixed point, at and after the first launch's end, in the third launch
@pytest.mark.parametrize("tol,most", [(1e-30, 1_000_000), (1e-30, 8192), (1e-30, 8193), (1e-30, 16389)])
def test_value_iteration_over_several_launches(mdpvi, tol, most):
    import torch
    p = _inst(3, 8, 2, 0.9997)
    V0 = torch.zeros(p.num_states, device="cuda")
    a, ia, ra = _vi(mdpvi, p, True, V0, tol, most)
    b, ib, rb = _vi(mdpvi, p, False, V0, tol, most)
    assert ia == ib and ra == rb and ia > 8191
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("tol,most", [(1e-10, 1_000_000), (1e-300, 8192), (1e-300, 8193), (1e-300, 16389)])
def test_evaluation_over_several_launches(mdpvi, tol, most):
    p = _inst(3, 8, 2, 0.999)
    a, ia, ra = _ev(mdpvi, p, True, tol, most)
    b, ib, rb = _ev(mdpvi, p, False, tol, most)
    assert ia > 8191 and (ia == ib or tol == 1e-10)
    stop = (ra + rb) * p.gamma / (1 - p.gamma) if ia != ib else 0.0   # both within their bound of the value
    assert float((a - b).abs().max()) <= _rounding(p) * float(b.abs().max()) + stop


@pytest.mark.parametrize("most", [1_000_000, 8193])
def test_batch_over_several_launches(mdpvi, most):
    import torch
    insts = [_inst(3, 8, 2, 0.9997), _inst(5, 9, 2, 0.9), _inst(4, 6, 3, 0.9), _inst(3, 5, 2, 0.9995)]
    b = mdpvi.Batch(insts)
    off = b.offsets
    V0 = torch.zeros(b.num_states, device="cuda")
    V0[off[2] + 1] = 0.25    # not invariant
    V = V0.clone()
    try:
        b.vi_solve(V, tol=1e-30, max_iter=most)
    except mdpvi.MdpviError as e:
        assert e.code == mdpvi.ENOCONV
    Ve = torch.zeros(b.num_states, dtype=torch.float64, device="cuda")
    pi = b.policy_greedy("least_loaded")
    ff = b.policy_greedy("first_fit")
    pi[off[2]:off[3]] = ff[off[2]:off[3]]
    try:
        b.policy_eval(pi, Ve, tol=1e-9, max_iter=most)
    except mdpvi.MdpviError as e:
        assert e.code == mdpvi.ENOCONV
    for i, p in enumerate(insts):
        sl = slice(off[i], off[i + 1])
        one, its, _ = _vi(mdpvi, p, False, V0[sl], 1e-30, most)
        assert torch.equal(one.view(torch.int32), V[sl].view(torch.int32)), i
        assert its > 8191 or i in (1, 2)
        mdp = mdpvi.MDP.from_instance(p)
        alone = torch.zeros(p.num_states, dtype=torch.float64, device="cuda")
        try:
            mdp.policy_eval(pi[sl].contiguous(), alone, tol=1e-9, max_iter=most)
        except mdpvi.MdpviError as e:
            assert e.code == mdpvi.ENOCONV
        assert torch.equal(alone, Ve[sl]), i


@pytest.mark.parametrize("C", [95, 113])
def test_the_most_lds(mdpvi, C):
    import torch
    p = _inst(2, C, 1, 0.9)
    V0 = torch.zeros(p.num_states, device="cuda")
    outs = [_vi(mdpvi, p, orbits, V0, 1e-6, 1_000_000) for orbits in (True, False)]
    assert outs[0][1:] == outs[1][1:] and torch.equal(outs[0][0], outs[1][0])
    a, ia, _ = _ev(mdpvi, p, True, 1e-300, 100)
    b, ib, _ = _ev(mdpvi, p, False, 1e-300, 100)
    assert ia == ib and float((a - b).abs().max()) <= _rounding(p) * float(b.abs().max())
    batch = mdpvi.Batch([p, _inst(3, 8, 2, 0.9)])
    V = torch.zeros(batch.num_states, device="cuda")
    batch.vi_solve(V, tol=1e-6)
    assert torch.equal(V[:p.num_states], outs[0][0])
    Ve = batch.policy_eval(batch.policy_greedy("least_loaded"), tol=1e-10)[0]
    assert torch.equal(Ve[:p.num_states], _ev(mdpvi, p, True, 1e-10, 1_000_000)[0])
