"""Value iteration on the orbits of the host permutations (automatic mode,
an invariant starting iterate) against the full sweeps of the direct form:
same bits, same sweep counts and residuals, at the edges of its launch
shapes; a starting iterate that is not invariant takes the full sweeps."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import sub_solution, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mdpvi():
    torch_cuda()
    import paper_2012_12419_amd as m
    m.load()
    return m


def _inst(K, C, J, **kw):
    size = [1 + j % C for j in range(J)]   # equal sizes where the classes outnumber the units
    return W.make(K, C, size, [0.7 / (1 + j) for j in range(J)], 0.1, 0.02, [1.1 * (1 + j) for j in range(J)],
                  kw.pop("gamma", 0.9), **kw)


# (K, C, J): one host; two; one wavefront; lanes per thread 1, 2 and more in
# the one-workgroup solve; 2, 4 and 8 lanes per orbit; the most hosts a digit
# byte packs and beyond (4-bit digits, 16-host loops); launched sweeps of one
# group per workgroup; 32-bit table entries
SHAPES = [(1, 1, 1), (1, 40, 3), (2, 9, 2), (2, 60, 1), (3, 5, 8), (4, 6, 5), (5, 5, 1), (5, 6, 3), (6, 4, 2),
          (8, 2, 2), (8, 3, 3), (9, 2, 2), (16, 1, 1), (12, 1, 1), (5, 9, 2), (4, 12, 3), (6, 7, 4)]


def _solve(mdpvi, p, form, V0, tol, max_iter=1_000_000):
    mdp = mdpvi.MDP.from_instance(p)
    mdp.set_sweep_form(form)
    V = V0.clone()
    try:
        st = mdp.vi_solve(V, tol=tol, max_iter=max_iter)
        code = 0
    except mdpvi.MdpviError as e:
        st, code = e.stats, e.code
    return V, st, code


@pytest.mark.parametrize("K,C,J", SHAPES)
@pytest.mark.parametrize("costs", [False, True])
def test_same_bits_as_full_sweeps(mdpvi, K, C, J, costs):
    import torch
    kw = dict(reject_cost=[0.2 + 0.1 * j for j in range(J)], idle_unit_cost=0.03) if costs else {}
    p = _inst(K, C, J, **kw)
    V0 = torch.full((p.num_states,), sub_solution(p), device="cuda")
    # to the fixed point; stopped in mid-chunk, at a chunk's end and just after it
    for tol, most in ((1e-6, 1_000_000), (1e-30, 17), (1e-30, 32), (1e-30, 33), (1e-30, 64)):
        a, sa, ca = _solve(mdpvi, p, 0, V0, tol, most)
        b, sb, cb = _solve(mdpvi, p, -1, V0, tol, most)
        assert ca == cb and sa["iterations"] == sb["iterations"], (most, sa, sb)
        assert sa["residual_inf"] == sb["residual_inf"]
        assert torch.equal(a.view(torch.int32), b.view(torch.int32)), most


def test_same_bits_with_wide_tables(mdpvi):
    # 74,613 orbits: table entries of 32 bits, several groups per workgroup
    import torch
    p = _inst(6, 16, 1, gamma=0.8)
    V0 = torch.zeros(p.num_states, device="cuda")
    a, sa, _ = _solve(mdpvi, p, 0, V0, 1e-3)
    b, sb, _ = _solve(mdpvi, p, -1, V0, 1e-3)
    assert sa["iterations"] == sb["iterations"] and sa["residual_inf"] == sb["residual_inf"]
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("K,C,J", [(3, 8, 2), (5, 9, 2)])
def test_other_starts(mdpvi, K, C, J):
    """A warm start from a solution (invariant), one state off it by an ulp
    in either half of the array (not invariant), and a NaN."""
    import torch
    p = _inst(K, C, J)
    sol, _, _ = _solve(mdpvi, p, -1, torch.zeros(p.num_states, device="cuda"), 1e-5)
    off = []
    for at in (1, p.num_states - 2):   # occupancies (1, 0, ..) and (C - 1, C, ..): others share their orbits
        V = sol.clone()
        V[at] = torch.nextafter(V[at], torch.tensor(1e9, device="cuda"))
        off.append(V)
    for V0 in [sol] + off:
        a, sa, _ = _solve(mdpvi, p, 0, V0, 1e-6)
        b, sb, _ = _solve(mdpvi, p, -1, V0, 1e-6)
        assert sa["iterations"] == sb["iterations"] and sa["residual_inf"] == sb["residual_inf"]
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    for V0 in (torch.full_like(sol, float("nan")), sol.clone()):
        V0[5] = float("nan")
        _, _, code = _solve(mdpvi, p, -1, V0, 1e-6)
        assert code == mdpvi.ENAN


def test_one_handle_many_calls(mdpvi):
    """A handle's orbit scratch serves later calls of other tolerances and
    starts, on another stream, and a refused call in between."""
    import torch
    p = _inst(5, 9, 2)
    mdp = mdpvi.MDP.from_instance(p)
    ref, _, _ = _solve(mdpvi, p, 0, torch.zeros(p.num_states, device="cuda"), 1e-6)
    side = torch.cuda.Stream()
    for k in range(3):
        V = torch.zeros(p.num_states, device="cuda")
        mdp.vi_solve(V, tol=1e-2)
        W_ = torch.rand(p.num_states, device="cuda")
        mdp.vi_solve(W_, tol=1e-3)
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            V.zero_()
            mdp.vi_solve(V, tol=1e-6, stream=side)
        torch.cuda.current_stream().wait_stream(side)
        assert torch.equal(V.view(torch.int32), ref.view(torch.int32)), k
