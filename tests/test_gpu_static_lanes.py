"""The lane-per-scenario form of the static kernels (from 32,768 scenarios)
against the wavefront-per-scenario form, which the same scenarios take in
smaller calls: every output, bit for bit, on the edges of the register
buckets (VCs), of the task chunks and of the last group of 64 scenarios, with
invalid scenarios among them (which leave everything but their status)."""
import numpy as np
import pytest

from tests.gpu_util import torch_cuda
from workloads import static_bot as ws

pytestmark = pytest.mark.gpu
B = 32768 + 37


@pytest.fixture(scope="module")
def mdpvi():
    torch_cuda()
    import paper_2012_12419_amd as m
    m.load()
    return m


@pytest.mark.parametrize("K,T", [(1, 0), (1, 7), (4, 63), (5, 64), (8, 65), (11, 55), (12, 128), (16, 129), (17, 3),
                                 (24, 40), (32, 64), (33, 70), (48, 66), (64, 130)])
def test_lanes_equal_wavefronts(mdpvi, K, T):
    import torch
    caps, need = ws.random_scenarios(B, K, T, seed=K * 131 + T, cap_max=40, need_max=9)
    rng = np.random.default_rng(K + T)
    place = rng.integers(-1, K, size=(B, T)).astype(np.int32)
    big = rng.choice(B, size=60, replace=False)
    caps[big[:10], rng.integers(0, K, 10)] = -1 - rng.integers(0, 5)
    caps[big[10:20], rng.integers(0, K, 10)] = (1 << 30) + 1
    caps[big[20:30]] = 1 << 30
    if T:
        need[big[30:40], rng.integers(0, T, 10)] = -3
        need[big[40:45], rng.integers(0, T, 5)] = (1 << 30) + 7
        need[big[20:30], :2] = 1 << 30
        place[big[45:50], rng.integers(0, T, 5)] = K
        place[big[50:55], rng.integers(0, T, 5)] = -7
        place[big[55:60]] = K - 1
        caps[big[55:60]] = 1 << 20
    c, n, p = (torch.from_numpy(x).cuda() for x in (caps, need, place))
    cut = [0, 16000, 32000, B]
    for call in (lambda a, b, q: mdpvi.static_first_fit(a, b), lambda a, b, q: mdpvi.static_score(a, b, q)):
        # outputs of invalid scenarios are not written: compared on the valid ones
        whole = call(c, n, p)
        parts = [call(c[i:j].contiguous(), n[i:j].contiguous(), p[i:j].contiguous()) for i, j in zip(cut, cut[1:])]
        ref = {k: torch.cat([x[k] for x in parts]) for k in whole}
        assert torch.equal(whole["status"], ref["status"])
        ok = ref["status"] == 0
        for k in whole:
            assert torch.equal(whole[k][ok], ref[k][ok]), k


def test_invalid_scenarios_write_only_their_status(mdpvi):
    import ctypes
    import torch
    K, T = 11, 70
    caps, need = ws.random_scenarios(B, K, T, seed=5)
    caps[::3, 2] = -1
    need[1::3, 69] = -1
    c, n = torch.from_numpy(caps).cuda(), torch.from_numpy(need).cuda()
    out = dict(place=torch.full((B, T), 77, dtype=torch.int32, device="cuda"),
               used=torch.full((B, K), 77, dtype=torch.int32, device="cuda"),
               totals=torch.full((B, 3), 77, dtype=torch.int64, device="cuda"),
               reward=torch.full((B,), 77.0, dtype=torch.float64, device="cuda"),
               status=torch.full((B,), 77, dtype=torch.int32, device="cuda"))
    ptr = {k: ctypes.c_void_p(v.data_ptr()) for k, v in out.items()}
    rc = mdpvi.load().static_first_fit(ctypes.c_void_p(c.data_ptr()), ctypes.c_void_p(n.data_ptr()), B, K, T, 1.0, 1.2,
                                       1.0, ptr["place"], ptr["used"], ptr["totals"], ptr["reward"], ptr["status"],
                                       None)
    torch.cuda.synchronize()
    assert rc == mdpvi.OK
    st = out["status"].cpu().numpy()
    assert np.all(st[::3] == 1) and np.all(st[1::3] == 2) and np.all(st[2::3] == 0)
    bad = torch.from_numpy(st != 0).cuda()
    for k in ("place", "used", "totals", "reward"):
        assert bool((out[k][bad] == 77).all()), k
        assert not bool((out[k][~bad] == 77).all()), k
