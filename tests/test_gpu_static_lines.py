"""Placing many scenarios of many VCs: on either side of the lines between the
forms (a wavefront or a lane per scenario), with the last register buckets of
the lane form, the same outputs as in calls of a few scenarios."""
import pytest

from tests.gpu_util import torch_cuda
from workloads import static_bot as ws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,T,line", [(24, 9, 32768), (25, 65, 49152), (32, 64, 49152), (33, 66, 163840),
                                      (48, 63, 163840), (49, 5, 163840)])
def test_lines_of_the_lane_form(K, T, line):
    torch = torch_cuda()
    import paper_2012_12419_amd as mdpvi
    caps, need = ws.random_scenarios(line + 37, K, T, seed=K + T, cap_max=9, need_max=6)
    c, n = torch.from_numpy(caps).cuda(), torch.from_numpy(need).cuda()
    cuts = list(range(0, line + 37, 20000)) + [line + 37]
    parts = [mdpvi.static_first_fit(c[i:j].contiguous(), n[i:j].contiguous()) for i, j in zip(cuts, cuts[1:])]
    ref = {k: torch.cat([x[k] for x in parts]) for k in parts[0]}
    for B in (line - 1, line, line + 37):
        got = mdpvi.static_first_fit(c[:B].contiguous(), n[:B].contiguous())
        for k in got:
            assert torch.equal(got[k], ref[k][:B]), (B, k)
