"""Scratch memory at its limits, on the host: the library runs in a process of
its own against a stand-in HIP runtime (fake_hip.c) whose allocations and
copies fail on demand.  Kernels do not run, so solves end with ENOCONV or ENAN;
what counts is the code, the kernels that would have been launched and the
memory held."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
f = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)
f.fake_log.restype = ctypes.c_char_p
f.fake_first_arg.restype = ctypes.c_void_p
for n in ("fake_live", "fake_peak"):
    getattr(f, n).restype = ctypes.c_size_t
f.fake_set_budget.argtypes = [ctypes.c_size_t]
import paper_2012_12419_amd as m
assert "torch" not in sys.modules
lib = m.load()
def params(K, C, J):
    return m.make_params(K, C, [1 + j for j in range(J)], [0.5] * J, 0.1, 0.02, [1.0 + j for j in range(J)], 0.9)
def handle(K, C, J):
    p, keep = params(K, C, J)
    h = ctypes.c_void_p()
    assert lib.mdp_build(ctypes.byref(p), ctypes.byref(h)) == m.OK
    return h
def batch(shapes):
    ps = [params(*s) for s in shapes]
    a = (m.Params * len(ps))(*[p for p, _ in ps])
    b = ctypes.c_void_p()
    assert lib.mdp_build_batch(a, len(ps), ctypes.byref(b)) == m.OK
    return b
V = ctypes.create_string_buffer(8 << 22)      # stands for every device array of a caller
pi = ctypes.create_string_buffer(1 << 22)
def log():
    return f.fake_log().decode()
def vi(h, it=40):
    return lib.vi_solve(h, V, 1e-6, it, None, None)
def ev(h, it=40):
    return lib.policy_eval(h, pi, V, 1e-6, it, None, None)
def vib(b, it=40):
    return lib.vi_solve_batch(b, V, 1e-6, it, None, None, None, None)
def evb(b, it=40):
    return lib.policy_eval_batch(b, pi, V, 1e-6, it, None, None, None, None)
RAN = (m.ENOCONV, m.ENAN)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not shutil.which("gcc"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("fake_hip")
    fake = str(d / "libamdhip64.so.7")
    vers = d / "versions"
    vers.write_text("hip_4.2 { *; };\nhip_4.3 { hipGraph*; };\nhip_6.0 { hipGetDeviceProperties*; };\n")
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7",
                    f"-Wl,--version-script={vers}", os.path.join(HERE, "fake_hip.c"), "-o", fake], check=True)

    def go(body):
        code = PRELUDE.format(root=ROOT, fake=fake) + body
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return go


def test_every_failed_allocation_of_a_handle_is_made_up_for(run):
    """Each allocation of the full sweeps fails once: ENOMEM, and the next call
    on the handle runs; nothing is left allocated."""
    run("""
before = f.fake_live()
for call in (vi, ev):
    for fail in (f.fake_fail_malloc, f.fake_fail_host):
        for n in range(20):
            f.fake_reset()
            h = handle(5, 10, 2)
            lib.mdp_set_orbits(h, 0)
            fail(n)
            rc = call(h)
            if rc in RAN:
                assert n >= 2
                break
            assert rc == m.ENOMEM, (n, rc, lib.mdpvi_last_error())
            assert call(h) in RAN, (n, lib.mdpvi_last_error())
            lib.mdp_free(h)
        else:
            raise AssertionError("never ran")
        lib.mdp_free(h)
assert f.fake_live() == before
""")


def test_a_failed_copy_of_the_model_is_made_again(run):
    """The evaluation sweeps read the model from device memory: after a failed
    copy the next call copies it again."""
    run("""
h = handle(4, 6, 2)
lib.mdp_set_orbits(h, 0)
f.fake_fail_copy(0)
assert ev(h) == m.EDEVICE
rc = ev(h)
assert rc in RAN, (rc, lib.mdpvi_last_error())
at = f.fake_first_arg(b"eval_exact_kernel")
K, C, J = ctypes.cast(at, ctypes.POINTER(ctypes.c_int32 * 3)).contents
assert (K, C, J) == (4, 6, 2)
""")


@pytest.mark.parametrize("call", ["vi", "ev"])
@pytest.mark.parametrize("shape", [(6, 7, 2), (8, 9, 1), (3, 8, 2)])
def test_orbit_tables_make_room_for_the_full_sweeps(run, call, shape):
    """A call that the orbit form refuses, on a device with just the memory
    that the full sweeps need, runs them."""
    run(f"""
shape, call = {shape}, {call}
V = ctypes.create_string_buffer(16 * shape[2] * (shape[1] + 1) ** shape[0])
pi = ctypes.create_string_buffer(shape[2] * (shape[1] + 1) ** shape[0])
h = handle(*shape)
lib.mdp_set_orbits(h, 0)
assert call(h) in RAN
need = f.fake_live()
lib.mdp_free(h)
for spare in (0, 4096, 1 << 16, 1 << 20):
    f.fake_reset()
    f.fake_refuse(1)
    f.fake_set_budget(need + spare)
    h = handle(*shape)
    for _ in range(3):
        assert call(h) in RAN, (spare, lib.mdpvi_last_error())
    lib.mdp_free(h)
    assert f.fake_live() == 0
""")


def test_a_solve_without_memory_for_the_tables_takes_the_full_sweeps(run):
    run("""
V = ctypes.create_string_buffer(8 * 3 * 11 ** 6)
for call, kernel in ((vi, "vi_tile_kernel"), (ev, "eval_tile_kernel")):
    f.fake_reset()
    h = handle(6, 10, 3)
    f.fake_fail_malloc(0)            # the tables are allocated first
    assert call(h) in RAN
    assert "orbit" not in log() and kernel in log()
    lib.mdp_free(h)
""")


SHAPES = "[(3, 8, 2), (4, 6, 3), (5, 9, 2), (6, 4, 2)]"


def test_batch_without_memory_for_its_plan_takes_the_full_forms(run):
    """A failed device or pinned allocation of the batch's orbit plan: the full
    forms run, and the plan is not tried again."""
    run(f"""
shapes = {SHAPES}
b = batch(shapes)
assert vib(b) != m.EDEVICE and "orbit_batch" in log()   # the plan's allocations: pinned, then device memory
lib.mdp_free_batch(b)
for which in (f.fake_fail_host, f.fake_fail_malloc):
    f.fake_reset()
    b = batch(shapes)
    lib.batch_set_orbits(b, 0)
    rc = vib(b)                      # the batch's own scratch
    lib.batch_set_orbits(b, -1)
    f.fake_reset()
    which(0)
    assert vib(b) == rc, lib.mdpvi_last_error()
    assert "orbit" not in log() and "batch_lds" in log()
    assert vib(b) == rc and "orbit" not in log()
    lib.mdp_free_batch(b)
assert f.fake_live() == 0
""")


def test_batch_plan_makes_room_for_later_scratch(run):
    """The evaluation's FP64 scratch, allocated after a value iteration on
    orbits, on a device with just the memory that the full forms need."""
    run(f"""
shapes = {SHAPES}
b = batch(shapes)
lib.batch_set_orbits(b, 0)
vib(b)
rc = evb(b)
need = f.fake_live()
lib.mdp_free_batch(b)
f.fake_reset()
b = batch(shapes)
vib(b)
assert "orbit_batch" in log()
with_plan = f.fake_live()
f.fake_set_budget(max(need, with_plan))
assert with_plan + 8 * lib.batch_num_states(b, -1) > max(need, with_plan)
assert evb(b) == rc, lib.mdpvi_last_error()
lib.mdp_free_batch(b)
assert f.fake_live() == 0
""")
