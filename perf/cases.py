"""Timed cases of the placement solver: what a program that uses the package
asks of it, through the package's own entry points.

A capacity planner solves one fleet (value iteration, then the greedy
policy), scores the fast heuristic beside it, differentiates the expected
reward with respect to the rates, and sweeps hundreds of uneven parameter
sets in one batch; the static example places one-shot bags of tasks.  Sizes
follow the package's workloads (1,458 to 58 million states, batches of 2 to
5 hosts of 4 to 12 units) and `draw` spreads over the ranges between them.

`exact` recomputes a case in 64 bits over the whole state space with plain
torch, without the package.
"""
import math

import numpy as np
import torch

import paper_2012_12419_amd as mdpvi
from paper_2012_12419_amd.autograd import expected_reward
import workloads as W

DEV = "cuda"


def listed():
    return [
        # the smallest call a planner makes: one small fleet, launches and latency
        dict(name="vi_small", kind="vi", K=3, C=8, J=2, gamma=0.95, tol=1e-6, reject=0.0, idle=0.0),
        # an ordinary fleet with every option of the reward: paid-cloud costs, idle penalty
        dict(name="vi_costs_mid", kind="vi", K=4, C=12, J=3, gamma=0.97, tol=1e-6, reject=0.3, idle=0.02),
        # the package's large single instance
        dict(name="vi_large", kind="vi", K=6, C=10, J=3, gamma=0.99, tol=1e-6, reject=0.0, idle=0.0),
        # one host more: beyond the last-level cache
        dict(name="vi_beyond_cache", kind="vi", K=7, C=10, J=3, gamma=0.99, tol=1e-6, reject=0.0, idle=0.0),
        # scoring the fast heuristic (least-loaded host) of the large instance in FP64
        dict(name="heuristic_large", kind="heuristic", rule="least_loaded", K=6, C=10, J=3, gamma=0.99, tol=1e-10),
        # scoring the paper's first-fit rule on an ordinary fleet
        dict(name="heuristic_first_fit", kind="heuristic", rule="first_fit", K=4, C=12, J=3, gamma=0.97, tol=1e-10),
        # the greedy policy and its gaps of a value function in hand
        dict(name="extract_large", kind="extract", dtype="f32", gap=True, K=6, C=10, J=3, gamma=0.99),
        # a training step on the rates: optimal reward and its gradient through autograd
        dict(name="gradient_step", kind="gradient", K=5, C=10, J=2, gamma=0.98),
        # sensitivities of one fixed policy: the adjoint alone
        dict(name="adjoint_mid", kind="adjoint", K=5, C=8, J=3, gamma=0.97),
        # the parameter sweep: hundreds of uneven fleets in one call
        dict(name="batch_vi", kind="batch_vi", n=512, tol=1e-6),
        # the sweep's gradients and heuristic scores
        dict(name="batch_gradient", kind="batch_gradient", n=128),
        # one-shot bags of tasks, a million scenarios of the published example's shape
        dict(name="static_bags", kind="static", op="first_fit", n=1_000_000, K=11, T=55),
    ]


def draw(rng):
    kind = rng.choice(["vi", "vi", "heuristic", "extract", "gradient", "adjoint", "batch_vi", "batch_gradient",
                       "static"])
    if kind == "batch_vi":
        return dict(kind=kind, n=int(round(8 * 64 ** rng.random())), tol=rng.choice([1e-6, 1e-5, 1e-4]))
    if kind == "batch_gradient":
        return dict(kind=kind, n=int(round(8 * 16 ** rng.random())))
    if kind == "static":
        return dict(kind=kind, op=rng.choice(["first_fit", "score"]), n=int(round(100 * 1e4 ** rng.random())),
                    K=rng.randint(2, 40), T=rng.randint(5, 80))
    # one instance: hosts, capacity and classes at random within the kind's states
    most = {"vi": 3e7, "heuristic": 5.4e6, "extract": 3e7, "gradient": 4e5, "adjoint": 1.5e6}[kind]
    target = 500.0 * (most / 500.0) ** rng.random()
    J = rng.randint(1, 4)
    K = rng.randint(2, 7)
    C = int((target / J) ** (1.0 / K)) - 1
    C = max(J, min(24, C))
    while J * (C + 1) ** K > most and K > 2:
        K -= 1
    case = dict(kind=kind, K=K, C=C, J=J, gamma=round(rng.uniform(0.9, 0.99), 4))
    if kind == "vi":
        case.update(tol=rng.choice([1e-6, 1e-5, 1e-4]), reject=rng.choice([0.0, 0.0, 0.3]),
                    idle=rng.choice([0.0, 0.0, 0.02]))
    elif kind == "heuristic":
        case.update(rule=rng.choice(["least_loaded", "first_fit"]), tol=rng.choice([1e-9, 1e-10]))
    elif kind == "extract":
        case.update(dtype=rng.choice(["f32", "f64"]), gap=rng.random() < 0.5)
    return case


# ------------------------------------------------------------------ inputs


def _rates(rng, K, C, J, gamma, load=None, reject=0.0, idle=0.0):
    """One parameter set: the rates of the package's workloads.  `load` scales
    the arrivals to that share of the capacity, so that placement matters."""
    lam = rng.uniform(0.2, 1.0, size=J)
    mu = rng.uniform(0.05, 0.2)
    nu = rng.uniform(0.005, 0.05)
    size = np.arange(1, J + 1)
    if load is not None:
        lam = lam * (load * rng.uniform(0.9, 1.1) * K * C * mu / float(lam @ size))
    reward = size * rng.uniform(0.8, 1.2, size=J)
    cost = rng.uniform(0.5, 1.0, size=J) * reject
    return W.make(K, C, size, lam, mu, nu, reward, gamma, reject_cost=cost, idle_unit_cost=idle)


def _instance(case, seed):
    rng = np.random.default_rng(seed)
    load = 1.2 if case["kind"] == "gradient" else None
    p = _rates(rng, case["K"], case["C"], case["J"], case["gamma"], load, case.get("reject", 0.0),
               case.get("idle", 0.0))
    if case["kind"] == "gradient":   # parameters of a torch program: float32
        p = p.replace(lam=np.float32(p.lam).tolist(), mu=float(np.float32(p.mu)), nu=float(np.float32(p.nu)),
                      reward=np.float32(p.reward).tolist())
    return p


def _instances(case, seed):
    # the shapes of the package's parameter sweep, other rates with each seed
    rng = np.random.default_rng(seed)
    return [_rates(rng, p.K, p.C, p.J, p.gamma) for p in W.batch(case["n"], seed=3)]


def _start(p):
    """The constant sub-solution that value iteration increases from: 0 where
    nothing costs, else the least one-step reward over the horizon."""
    Lam = sum(p.lam) + p.K * p.C * p.mu + p.K * p.nu
    return -(sum(p.lam) / Lam * max(p.reject_cost) + p.idle_unit_cost * p.K * p.C) / (1 - p.gamma)


def _value_in_hand(p, seed):
    """A value function as a solver or an approximation of it leaves one: it
    falls with every unit in use, faster on a fuller host, with a small
    part of its own at each state."""
    R, n_occ = p.C + 1, (p.C + 1) ** p.K
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed + 1)
    a, b = rng.uniform(0.05, 0.1), rng.uniform(0.002, 0.01)
    V = torch.empty(p.J, n_occ, dtype=torch.float64, device=DEV)
    o = torch.arange(n_occ, device=DEV)
    load = torch.zeros(n_occ, dtype=torch.float64, device=DEV)
    for _ in range(p.K):
        d = (o % R).double()
        load += a * d + b * d * d
        o = o // R
    for e in range(p.J):
        V[e] = 50.0 + 0.3 * e - load * (1 + 0.02 * e)
    V += 1e-3 * torch.rand(V.shape, generator=gen, dtype=torch.float64, device=DEV)
    return V.reshape(-1)


def _scenarios(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n, K, T = case["n"], case["K"], case["T"]
    caps = torch.randint(0, 46, (n, K), generator=gen, device=DEV, dtype=torch.int32)
    need = torch.randint(1, 12, (n, T), generator=gen, device=DEV, dtype=torch.int32)
    need[torch.rand((n, T), generator=gen, device=DEV) < 0.1] = 0
    length = torch.randint(T // 2, T + 1, (n, 1), generator=gen, device=DEV)
    need[torch.arange(T, device=DEV)[None, :] >= length] = 0
    return caps, need


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case)
    if kind == "static":
        s["caps"], s["need"] = _scenarios(case, seed)
        if case["op"] == "score":
            # a placement from elsewhere: each task on the VC that a hash of its slot names, paid where that is full
            s["place"] = _round_robin(s["caps"], s["need"])
        return s
    if kind in ("batch_vi", "batch_gradient"):
        insts = _instances(case, seed)
        s["batch"] = mdpvi.Batch(insts)
        s["J_sizes"] = [p.J for p in insts]
        return s
    p = _instance(case, seed)
    if kind == "gradient":
        s["inst"] = p
        s["theta"] = [torch.tensor(x, dtype=torch.float32, requires_grad=True) for x in
                      (p.lam, p.mu, p.nu, p.reward)]
        return s
    s["mdp"] = mdpvi.MDP.from_instance(p)
    s["start"] = _start(p)
    if kind == "extract":
        V = _value_in_hand(p, seed)
        s["V"] = V if case["dtype"] == "f64" else V.float()
    elif kind == "adjoint":
        s["pi"] = s["mdp"].policy_greedy("least_loaded")
        s["V_pi"], _ = s["mdp"].policy_eval(s["pi"], tol=1e-11)
    return s


def _round_robin(caps, need):
    n, K = caps.shape
    left = caps.clone()
    place = torch.full_like(need, mdpvi.STATIC_EMPTY)
    rows = torch.arange(n, device=caps.device)
    for t in range(need.shape[1]):
        k = (rows + 7 * t) % K
        want = need[:, t]
        room = (left[rows, k] >= want) & (want > 0)
        left[rows, k] -= torch.where(room, want, torch.zeros_like(want))
        place[:, t] = torch.where(want == 0, torch.full_like(want, mdpvi.STATIC_EMPTY),
                                  torch.where(room, k.to(torch.int32), torch.full_like(want, mdpvi.STATIC_PAID)))
    return place


# -------------------------------------------------------------------- passes


def run(s):
    kind = s["kind"]
    if kind == "vi":
        V = torch.full((s["mdp"].num_states,), s["start"], dtype=torch.float32, device=DEV)
        s["mdp"].vi_solve(V, tol=s["tol"])
        return {"V": V}
    if kind == "heuristic":
        pi = s["mdp"].policy_greedy(s["rule"])
        V, _ = s["mdp"].policy_eval(pi, tol=s["tol"])
        return {"pi": pi, "V": V}
    if kind == "extract":
        pi, gap = s["mdp"].policy_extract(s["V"], want_gap=s["gap"])
        return {"pi": pi, "gap": gap} if s["gap"] else {"pi": pi}
    if kind == "gradient":
        p = s["inst"]
        lam, mu, nu, reward = s["theta"]
        for t in s["theta"]:
            t.grad = None
        J = expected_reward(lam, mu, nu, reward, p.K, p.C, p.size, p.gamma)
        J.backward()
        return {"J": J.detach(), "lam": lam.grad, "mu": mu.grad, "nu": nu.grad, "reward": reward.grad}
    if kind == "adjoint":
        grad, J, w, _ = s["mdp"].vi_adjoint(s["pi"], s["V_pi"])
        return {"grad": torch.tensor(grad), "J": J, "w": w}
    if kind == "batch_vi":
        V = torch.zeros(s["batch"].num_states, dtype=torch.float32, device=DEV)
        s["batch"].vi_solve(V, tol=s["tol"])
        return {"V": V}
    if kind == "batch_gradient":
        b = s["batch"]
        V = torch.zeros(b.num_states, dtype=torch.float32, device=DEV)
        b.vi_solve(V, tol=1e-6)
        pi, _ = b.policy_extract(V, want_gap=False)
        Vp = V.double()
        b.policy_iteration(pi, Vp, eval_tol=1e-12, improve_tol=1e-9)
        grads, objs, _, _, _ = b.vi_adjoint(pi, Vp, s["J_sizes"])
        greedy = b.policy_greedy("least_loaded")
        Vg, _, _, _ = b.policy_eval(greedy, Vp.clone())
        return {"V_opt": Vp, "V_greedy": Vg, "greedy": greedy, "J": torch.tensor(objs, dtype=torch.float64),
                "grad": torch.tensor([x for g in grads for x in g])}
    if s["op"] == "first_fit":
        return mdpvi.static_first_fit(s["caps"], s["need"])
    return mdpvi.static_score(s["caps"], s["need"], s["place"])


# ---------------------------------------------------------------------- work


def _shapes(case):
    if "K" in case:
        return [(case["K"], case["C"], case["J"], case["gamma"])]
    return [(p.K, p.C, p.J, p.gamma) for p in W.batch(case["n"], seed=3)]


def work(case):
    """Bytes: every per-state array read or written once per call.  Operations:
    one backup of every state per sweep (2 K + 2 multiply-adds and K
    comparisons), the sweeps that a discount needs to reach the tolerance."""
    kind = case["kind"]
    if kind == "static":
        n, K, T = case["n"], case["K"], case["T"]
        return {"bytes": n * (4.0 * K + 8 * T + 4 * K + 24 + 8 + 4), "flops": 2.0 * n * T}
    tol = {"gradient": 1e-6, "adjoint": 1e-10, "batch_gradient": 1e-12}.get(kind, case.get("tol", 1e-6))
    out = {"bytes": 0.0, "flops": 0.0}
    for K, C, J, gamma in _shapes(case):
        N = J * (C + 1.0) ** K
        sweeps = 1.0 if kind == "extract" else math.log(tol) / math.log(gamma)
        per = {"vi": 8, "heuristic": 17, "extract": 9 if case.get("dtype") == "f64" else 5, "gradient": 25,
               "adjoint": 17, "batch_vi": 8, "batch_gradient": 34}[kind]
        if case.get("gap"):
            per += 4
        out["bytes"] += per * N
        out["flops"] += N * (5.0 * K + 6) * sweeps
    return out


# --------------------------------------------------------------------- exact


class Whole:
    """One instance in 64 bits over the whole state space: values as a tensor
    [J, R, .., R] whose last axis is host 0's occupancy."""

    def __init__(self, p):
        self.p, self.K, self.J, self.R = p, p.K, p.J, p.C + 1
        self.occ = (self.R,) * self.K
        lam = torch.tensor(p.lam, dtype=torch.float64, device=DEV)
        self.theta = [lam, torch.tensor(p.mu, dtype=torch.float64, device=DEV),
                      torch.tensor(p.nu, dtype=torch.float64, device=DEV),
                      torch.tensor(p.reward, dtype=torch.float64, device=DEV)]
        d = torch.arange(self.R, dtype=torch.float64, device=DEV)
        self.digit = [d.reshape((1,) * (self.K - 1 - k) + (self.R,) + (1,) * k) for k in range(self.K)]
        self.free = sum(p.C - x for x in self.digit).expand(self.occ)

    def rates(self):
        lam, mu, nu, r = self.theta
        Lam = lam.sum() + self.K * self.p.C * mu + self.K * nu
        cost = torch.tensor(self.p.reject_cost, dtype=torch.float64, device=DEV)
        P = lam.sum() / Lam
        return lam / Lam, mu / Lam, nu / Lam, P * r, -P * cost

    def stay(self, V, mu_L, nu_L):
        """The part of P V that no decision changes: releases, resets, idling."""
        J, K = self.J, self.K
        D = self.free * V * mu_L
        for k in range(K):
            ax = K - k
            n = V.shape[ax]
            D.narrow(ax, 1, n - 1).add_(V.narrow(ax, 0, n - 1) * (mu_L * self.digit[k].narrow(K - 1 - k, 1, n - 1)))
            D.add_(V.narrow(ax, 0, 1) * nu_L)
        return D

    def placed(self, A, e, k):
        """A at the occupancy with size_e units more on host k, -inf where it has no room."""
        out = torch.full_like(A, -math.inf)
        ax, s = self.K - 1 - k, self.p.size[e]
        out.narrow(ax, 0, self.R - s).copy_(A.narrow(ax, s, self.R - s))
        return out

    def q(self, V, e, D, pl, rates):
        """(best Q of a placement on host k, for each k) and the paid cloud's."""
        p_j, _, _, place, paid = rates
        A = (V * p_j.reshape((-1,) + (1,) * self.K)).sum(0)
        hold = self.p.idle_unit_cost * self.free
        qs = [place[e] - hold + pl * (self.placed(A, e, k) + D[e]) for k in range(self.K)]
        qs.append(paid[e] - hold + pl * (A + D[e]))
        return qs

    def optimal(self, V, tol):
        rates = self.rates()
        p_j, mu_L, nu_L, place, paid = rates
        g = self.p.gamma
        w = p_j.reshape((-1,) + (1,) * self.K)
        hold = self.p.idle_unit_cost * self.free
        for i in range(100000):
            A = (V * w).sum(0)
            new = self.stay(V, mu_L, nu_L)
            for e in range(self.J):
                best = torch.full_like(A, -math.inf)
                s = self.p.size[e]
                for k in range(self.K):
                    ax = self.K - 1 - k
                    t = best.narrow(ax, 0, self.R - s)
                    torch.maximum(t, A.narrow(ax, s, self.R - s), out=t)
                new[e].add_(torch.maximum(best + place[e] / g, A + paid[e] / g))
            new.mul_(g).sub_(hold)
            if i % 16 == 15 and float((new - V).abs().max()) < tol:
                return new
            V = new
        return V

    def targets(self, pi):
        """Per state: the occupancy its arrival leads to, and whether it is placed."""
        n_occ = self.R ** self.K
        o = torch.arange(n_occ, device=DEV)
        stride = torch.tensor([self.R ** k for k in range(self.K)] + [0], device=DEV)
        act = pi.reshape(self.J, n_occ).long()
        size = torch.tensor(self.p.size, device=DEV)[:, None]
        return o[None, :] + size * stride[act], act < self.K

    def policy_backup(self, V, to, placed, rates):
        p_j, mu_L, nu_L, place, paid = rates
        A = (V.reshape(self.J, -1) * p_j[:, None]).sum(0)
        r = torch.where(placed, place[:, None], paid[:, None]).reshape(V.shape)
        D = self.stay(V, mu_L, nu_L) + A[to].reshape(V.shape)
        return r - self.p.idle_unit_cost * self.free + self.p.gamma * D

    def evaluate(self, pi, V, tol):
        to, placed = self.targets(pi)
        rates = self.rates()
        for i in range(100000):
            new = self.policy_backup(V, to, placed, rates)
            if i % 16 == 15 and float((new - V).abs().max()) < tol:
                return new
            V = new
        return V

    def zeros(self):
        return torch.zeros((self.J,) + self.occ, dtype=torch.float64, device=DEV)

    def greedy(self, V):
        """The best action of every state, the lowest index within rounding of it."""
        rates = self.rates()
        D = self.stay(V, rates[1], rates[2])
        out = []
        for e in range(self.J):
            q = torch.stack(self.q(V, e, D, self.p.gamma, rates))
            best = q.max(0).values
            out.append((q >= best - 1e-10 * best.abs()).to(torch.uint8).argmax(0))
        return torch.stack(out)

    def rule(self, kind):
        n = torch.stack([x.expand(self.occ) for x in self.digit])
        out = []
        for e in range(self.J):
            room = n + self.p.size[e] <= self.p.C
            if kind == "least_loaded":
                key = torch.where(room, n, torch.full_like(n, math.inf))
                a = key.argmin(0)
            else:
                a = room.to(torch.uint8).argmax(0)
            out.append(torch.where(room.any(0), a, torch.full_like(a, self.K)))
        return torch.stack(out)

    def weights(self, pi, tol):
        """w = c + gamma P_pi^T w."""
        to, _ = self.targets(pi)
        p_j, mu_L, nu_L, _, _ = self.rates()
        c = self.zeros()
        c.reshape(self.J, -1)[:, 0] = self.theta[0] / self.theta[0].sum()
        w = c.clone()
        K = self.K
        for i in range(100000):
            new = self.free * w * mu_L
            for k in range(K):
                ax = K - k
                up = w.narrow(ax, 1, self.R - 1) * (mu_L * self.digit[k].narrow(K - 1 - k, 1, self.R - 1))
                new.narrow(ax, 0, self.R - 1).add_(up)
                new.narrow(ax, 0, 1).add_(w.sum(ax, keepdim=True) * nu_L)
            mass = torch.zeros(self.R ** K, dtype=torch.float64, device=DEV)
            mass.index_add_(0, to.reshape(-1), w.reshape(-1))
            new += mass.reshape((1,) + self.occ) * p_j.reshape((-1,) + (1,) * K)
            new.mul_(self.p.gamma).add_(c)
            if i % 16 == 15 and float((new - w).abs().sum()) < tol:
                return new
            w = new
        return w

    def gradient(self, pi, V, w):
        """(J, dJ/dlambda, dJ/dmu, dJ/dnu, dJ/dr) with the policy held fixed:
        the derivative of sum w (r_pi + gamma P_pi V) + sum c V(0, .)."""
        to, placed = self.targets(pi)
        for t in self.theta:
            t.requires_grad_(True)
        lam = self.theta[0]
        start = (lam / lam.sum() * V.reshape(self.J, -1)[:, 0]).sum()
        f = (w * self.policy_backup(V, to, placed, self.rates())).sum() + start
        g = torch.autograd.grad(f, self.theta)
        for t in self.theta:
            t.requires_grad_(False)
        return [start.detach()] + list(g)


def _cost(shapes, passes=1.0):
    """Seconds of torch that 64-bit sweeps of these shapes take on the card."""
    t = 0.0
    for K, C, J, gamma in shapes:
        N = J * (C + 1.0) ** K
        t += passes * math.log(1e-13 * (1 - gamma)) / math.log(gamma) * (
            (4 * K + J * K + 4 * J + 6) * 8e-6 + N * 8 * (5 * K + 6) / 3e12)
    return t


def exact(case, seed):
    kind = case["kind"]
    if kind == "static":
        return _exact_static(case, seed)
    passes = {"vi": 1.0, "heuristic": 1.0, "extract": 0.0, "gradient": 3.5, "adjoint": 2.5, "batch_vi": 1.0,
              "batch_gradient": 4.5}[kind]
    if _cost(_shapes(case), passes) > 15.0:
        return None
    if kind == "batch_vi":
        return {"V": torch.cat([Whole(p).optimal(Whole(p).zeros(), 1e-11).reshape(-1)
                                for p in _instances(case, seed)])}
    if kind == "batch_gradient":
        got = [_exact_gradient(p) for p in _instances(case, seed)]
        V_g = []
        for p, (m, V, _, _) in zip(_instances(case, seed), got):
            V_g.append(m.evaluate(m.rule("least_loaded"), V, 1e-13).reshape(-1))
        return {"V_opt": torch.cat([V.reshape(-1) for _, V, _, _ in got]), "V_greedy": torch.cat(V_g), "greedy": None,
                "J": torch.stack([g[0] for _, _, _, g in got]),
                "grad": torch.cat([torch.cat([x.reshape(-1) for x in g[1:]]) for _, _, _, g in got])}
    p = _instance(case, seed)
    m = Whole(p)
    if kind == "vi":
        return {"V": m.optimal(m.zeros() + _start(p), 1e-11).reshape(-1)}
    if kind == "heuristic":
        return {"pi": None, "V": m.evaluate(m.rule(case["rule"]), m.zeros(), 1e-13).reshape(-1)}
    if kind == "extract":
        if not case["gap"]:
            return None
        V = _value_in_hand(p, seed)
        V = (V if case["dtype"] == "f64" else V.float().double()).reshape((p.J,) + m.occ)
        rates = m.rates()
        D = m.stay(V, rates[1], rates[2])
        gap = []
        for e in range(p.J):
            top = torch.stack(m.q(V, e, D, p.gamma, rates)).topk(2, 0).values
            gap.append(top[0] - top[1])
        return {"pi": None, "gap": torch.stack(gap).reshape(-1)}
    if kind == "gradient":
        _, _, _, g = _exact_gradient(p)
        return dict(zip(("J", "lam", "mu", "nu", "reward"), (x.cpu() for x in g)))
    pi = m.rule("least_loaded")
    V = m.evaluate(pi, m.zeros(), 1e-13)
    w = m.weights(pi, 1e-13)
    g = m.gradient(pi, V, w)
    return {"grad": torch.cat([x.reshape(-1) for x in g[1:]]).cpu(), "J": float(g[0]), "w": w.reshape(-1)}


def _exact_gradient(p):
    m = Whole(p)
    V = m.optimal(m.zeros() + _start(p), 1e-12)
    pi = m.greedy(V)
    V = m.evaluate(pi, V, 1e-13)
    w = m.weights(pi, 1e-13)
    return m, V, pi, m.gradient(pi, V, w)


def _exact_static(case, seed):
    caps, need = _scenarios(case, seed)
    left = caps.long()
    place = _round_robin(caps, need) if case["op"] == "score" else None
    n, K = caps.shape
    rows = torch.arange(n, device=DEV)
    vc = torch.zeros(n, dtype=torch.int64, device=DEV)
    paid = torch.zeros_like(vc)
    for t in range(need.shape[1]):
        want = need[:, t].long()
        if place is None:
            room = left >= want[:, None]
            k = room.to(torch.uint8).argmax(1)
            on = room.any(1) & (want > 0)
        else:
            k = place[:, t].long().clamp(min=0)
            on = (place[:, t] >= 0) & (want > 0)
        took = torch.where(on, want, torch.zeros_like(want))
        left[rows, k] -= took
        vc += took
        paid += want - took
    reward = vc.double() - 1.2 * paid.double() - left.sum(1).double()
    out = {"used": None, "totals": None, "reward": reward, "status": None}
    if place is None:
        out["place"] = None
    return out
