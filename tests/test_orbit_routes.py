"""What a solve launches, in order, on the host against the stand-in HIP runtime
(fake_hip.c; no kernel runs, so no solve stops before max_iter): short calls
take as little as without the orbit form."""
import pytest

from tests.test_scratch_limits import run  # noqa: F401  (the fixture)

SHAPE = """
def steps(call):
    f.fake_reset()
    call()
    names = []
    for l in log().split("\\n"):
        for part, short in (("orbit_check", "check"), ("orbit_verdict", "verdict"), ("orbit_sweep", "orbit"),
                            ("orbit_lds", "lds"), ("orbit_expand", "expand"), ("hipGraphInstantiate", "record"),
                            ("hipGraphLaunch", "chunk"), ("eval_exact", "full"), ("eval_tile", "full"),
                            ("vi_exact", "full"), ("vi_tile", "full"), ("vi_arrival", "full")):
            if part in l and not (part == "orbit_verdict" and "check" in l):
                names.append(short)
                break
    out = []
    for n in names:
        if out and out[-1][0] == n:
            out[-1][1] += 1
        else:
            out.append([n, 1])
    return [tuple(x) for x in out]
"""


def test_short_value_iteration_is_full_sweeps(run):
    """Below a million states: 24 full sweeps before anything of the orbit form;
    at 5.3 million, and where one workgroup solves it, the check first."""
    run(SHAPE + """
got = steps(lambda: vi(handle(4, 12, 3), 100))
assert got[0] == ("full", 24) and got[1][0] == "check" and got[2][0] == "verdict", got
got = steps(lambda: vi(handle(4, 12, 3), 24))
assert got == [("full", 24)], got
V = ctypes.create_string_buffer(4 * 3 * 11 ** 6)
got = steps(lambda: vi(handle(6, 10, 3), 100))
assert got[:3] == [("check", 1), ("verdict", 1), ("orbit", 24)], got
got = steps(lambda: vi(handle(3, 8, 2), 100))
assert got == [("check", 1), ("lds", 1), ("expand", 1)], got
""")


def test_a_handles_first_solve_records_late(run):
    """Eight launched sweeps, waited for, then sixteen; only then the recording
    of a chunk, which later solves find."""
    run(SHAPE + """
h = handle(5, 9, 2)
got = steps(lambda: ev(h, 100))
assert got[:5] == [("check", 1), ("verdict", 1), ("orbit", 24), ("record", 1), ("chunk", 2)], got
got = steps(lambda: ev(h, 100))
assert got[:4] == [("check", 1), ("verdict", 1), ("orbit", 8), ("chunk", 2)], got
""")


@pytest.mark.parametrize("shape", [(5, 9, 2), (4, 12, 3)])
def test_a_refused_evaluation_adds_its_check(run, shape):
    """The check stands for the one of the policy's actions: beside the full
    sweeps a refused evaluation launches nothing else."""
    run(SHAPE + f"""
h = handle(*{shape})
lib.mdp_set_orbits(h, 0)
plain = steps(lambda: ev(h, 40))
lib.mdp_set_orbits(h, -1)
f.fake_reset()
ev(h, 40)
def refused():
    f.fake_refuse(1)
    ev(h, 40)
got = steps(refused)
assert got == [("check", 1), ("verdict", 1)] + plain, (got, plain)
""")
