"""Solves that stop at given sweeps: around the ends of the first chunks, the
sweep from which the full evaluation sweeps and the batch rounds leave the stop
test to one workgroup (32), and the sweep at which value iteration goes from the
full sweeps to the orbits (24).  The tolerance lies between the residuals of
two sweeps; the answer is the iterate of that many sweeps, bit for bit."""
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


STOPS = (1, 2, 7, 8, 9, 16, 22, 23, 24, 25, 26, 31, 32, 33, 34, 40, 55, 56, 57)


def _stops(mdpvi, solve):
    """solve(tol, max_iter) -> (array, stats) or raises; each stop's iterate and
    residual from a call with as many sweeps, then the call that stops there."""
    import torch

    def at(m):
        with pytest.raises(mdpvi.MdpviError) as e:
            solve(1e-300, m)
        assert e.value.code == mdpvi.ENOCONV
        return solve.array.clone(), e.value.stats["residual_inf"]

    for m in STOPS:
        V, r = at(m)
        before = at(m - 1)[1] if m > 1 else 2 * r
        if not r < before:
            continue
        st = solve(0.5 * (r + before), 1_000_000)
        assert st["iterations"] == m and st["residual_inf"] == r, m
        assert torch.equal(solve.array, V), m


class _Solve:
    def __init__(self, V0, call):
        self.V0, self.call, self.array = V0, call, None

    def __call__(self, tol, most):
        self.array = self.V0.clone()
        return self.call(self.array, tol, most)


# in LDS, with full sweeps first, orbits from the start (32^4 states and more), refused ones of all three
@pytest.mark.parametrize("K,C,J", [(3, 8, 2), (5, 9, 2), (4, 31, 1)])
@pytest.mark.parametrize("invariant", [True, False])
def test_value_iteration_stops(mdpvi, K, C, J, invariant):
    import torch
    p = _inst(K, C, J, gamma=0.8)
    mdp = mdpvi.MDP.from_instance(p)
    V0 = torch.zeros(p.num_states, device="cuda")
    if not invariant:
        V0[1] = 0.5
    solve = _Solve(V0, lambda V, tol, most: mdp.vi_solve(V, tol=tol, max_iter=most))
    _stops(mdpvi, solve)
    full = mdpvi.MDP.from_instance(p)
    full.set_orbits(False)
    for tol in (1e-2, 1e-4):
        a, b = V0.clone(), V0.clone()
        sa, sb = mdp.vi_solve(a, tol=tol), full.vi_solve(b, tol=tol)
        assert sa["iterations"] == sb["iterations"] and sa["residual_inf"] == sb["residual_inf"]
        assert torch.equal(a, b)


# exact-shape direct, tile and generic full sweeps; orbits in LDS and launched
@pytest.mark.parametrize("K,C,J,rule", [(4, 6, 3, "first_fit"), (4, 16, 1, "first_fit"), (9, 2, 2, "first_fit"),
                                        (3, 8, 2, "least_loaded"), (5, 9, 2, "least_loaded")])
def test_evaluation_stops(mdpvi, K, C, J, rule):
    import torch
    p = _inst(K, C, J, gamma=0.8)
    mdp = mdpvi.MDP.from_instance(p)
    pi = mdp.policy_greedy(rule)
    V0 = torch.zeros(p.num_states, dtype=torch.float64, device="cuda")
    # one orbit solve takes full sweeps below 32, which round otherwise: orbits in every call or in none
    solve = _Solve(V0, lambda V, tol, most: mdp.policy_eval(pi, V, tol=tol, max_iter=most)[1])
    if rule == "first_fit":
        _stops(mdpvi, solve)
    else:
        for tol in (0.3, 0.1, 1e-2, 1e-3, 1e-6):
            a = V0.clone()
            st = mdp.policy_eval(pi, a, tol=tol)[1]
            if st["iterations"] >= 32:
                with pytest.raises(mdpvi.MdpviError) as e:
                    b = V0.clone()
                    mdp.policy_eval(pi, b, tol=1e-300, max_iter=st["iterations"])
                assert e.value.code == mdpvi.ENOCONV and e.value.stats["residual_inf"] == st["residual_inf"]
                assert torch.equal(a, b)


@pytest.mark.parametrize("op", ["vi", "eval", "adjoint"])
def test_batch_rounds_stop(mdpvi, op):
    """Each instance of a batch of full rounds stops as it does alone, and as in
    a batch that stops it there by max_iter."""
    import torch
    insts = [_inst(5, 6, 3, 0.55), _inst(4, 12, 3, 0.8), _inst(5, 9, 2, 0.9), _inst(6, 4, 2, 0.7)]
    b = mdpvi.Batch(insts)
    b.set_orbits(False)
    off = b.offsets
    pi = b.policy_greedy("first_fit")
    n = b.num_states
    f64, f32 = (lambda: torch.zeros(n, dtype=torch.float64, device="cuda")), (lambda: torch.zeros(n, device="cuda"))
    Vp = b.policy_eval(pi, tol=1e-10)[0]

    def run(tol, most):
        if op == "vi":
            V = f32()
            return V, lambda: b.vi_solve(V, tol=tol, max_iter=most)[1]
        if op == "eval":
            V = f64()
            return V, lambda: b.policy_eval(pi, V, tol=tol, max_iter=most)[2]
        w = f32()
        return w, lambda: b.vi_adjoint(pi, Vp, [p.J for p in insts], w=w, tol=tol, max_iter=most)[4]

    seen = set()
    for tol in (0.5, 0.2, 0.1, 0.05, 0.02, 1e-2, 3e-3, 1e-3, 1e-4):
        X, call = run(tol, 1_000_000)
        its = call()
        for i, m in enumerate(its):
            seen.add(m)
            Y, cut = run(1e-300, m)
            with pytest.raises(mdpvi.MdpviError) as e:
                cut()
            assert e.value.code == mdpvi.ENOCONV
            assert torch.equal(X[off[i]:off[i + 1]], Y[off[i]:off[i + 1]]), (tol, i, m)
    assert min(seen) < 32 < max(seen)
