"""What the library's host code launches, read without a GPU: the library runs on
a HIP runtime of the host (tests/host_hip.cpp), in a process of its own."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2603_11045_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
hip.host_hip_launches.restype = ctypes.c_char_p
hip.host_hip_bytes.restype = ctypes.c_size_t
VP, D = ctypes.c_void_p, ctypes.c_double
lib.nh_create.argtypes = [VP, ctypes.c_int, VP]
lib.nh_set_grid.argtypes = [VP, ctypes.c_int, ctypes.c_int, ctypes.c_int, D, D, D]
lib.nh_set_launch.argtypes = [VP, ctypes.c_int, ctypes.c_int, ctypes.c_int]
lib.nh_set_cg_variant.argtypes = [VP, ctypes.c_int]
lib.nh_set_jacobi_sweeps.argtypes = [VP, ctypes.c_int]
lib.nh_set_boundary.argtypes = [VP, ctypes.c_int, D]
for f in (lib.nh_forward, lib.nh_forward_f64):
    f.argtypes = [VP, VP, VP, VP, D, ctypes.c_int, VP]
for f in (lib.nh_adjoint, lib.nh_adjoint_f64):
    f.argtypes = [VP, VP, VP]

ctx = VP()
assert lib.nh_create(ctypes.byref(ctx), 0, None) == 0

def grid(nx, ny, nz):
    global cells, columns
    cells, columns = nx * ny * nz, nx * ny
    assert lib.nh_set_grid(ctx, nx, ny, nz, 1.0, 1.0, 1.0) == 0

def forward(nsteps, double=False):
    a, q, t, s = (ctypes.create_string_buffer(8 * n) for n in (cells, columns, nsteps, columns * nsteps))
    return (lib.nh_forward_f64 if double else lib.nh_forward)(ctx, a, q, t, 1.0, nsteps, s)

def adjoint(nsteps, double=False):
    g, G = (ctypes.create_string_buffer(8 * n) for n in (columns * nsteps, cells))
    return (lib.nh_adjoint_f64 if double else lib.nh_adjoint)(ctx, g, G)

def launches(*words):
    lines = hip.host_hip_launches().decode().splitlines()
    return [l for l in lines if not words or any(w in l for w in words)]

STEPS = ("brick_steps_kernel", "jacobi_steps_kernel", "jacobi_deep_kernel", "step_kernel", "resident_full_kernel")
CLEAR = "fill_kernelIyE"                     # of 64-bit words: slots, halo words, tagged iterates
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("g++ and the HIP headers are needed")
    so = str(tmp_path_factory.mktemp("hip") / "libhost_hip.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-o", so, os.path.join(ROOT, "tests", "host_hip.cpp")], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]

    def go(code, **env):
        r = subprocess.run([sys.executable, "-c", PRELUDE + code, so, _lib.LIB_PATH], capture_output=True, text=True,
                           timeout=120, env={**os.environ, **env})
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
        return r

    return go


@pytest.mark.parametrize("setup,words", [
    ("grid(16, 16, 8)", 2), ("grid(64, 33, 12)", 2), ("grid(64, 40, 8); double = True", 2),
    ("grid(64, 64, 16); lib.nh_set_jacobi_sweeps(ctx, 10)", 1),
    ("grid(40, 20, 24); lib.nh_set_jacobi_sweeps(ctx, 10)", 1),
], ids=["one-brick", "bricks", "bricks-f64", "fixed-k", "fixed-k-deep"])
def test_tagged_words_are_cleared_whenever_the_tags_come_round(run, setup, words):
    """Tags repeat after 256 launch numbers: whichever of them a queue of several
    steps starts with, the words are cleared once before the first launch of a new
    round (slots; with bricks the halo words too)."""
    run(f"""
double = False
{setup}
assert forward(12, double) == 0
hip.host_hip_reset()
for k in range(6):                           # some 300 numbers in all: one new round
    assert forward(24, double) == 0 and adjoint(24, double) == 0
assert len(launches(*STEPS)) == 24
cleared = launches(CLEAR)
assert len(cleared) == len(set(cleared)) == {words}, cleared
lines = launches(CLEAR, *STEPS)              # in one go, before a step
first = lines.index(cleared[0])
assert lines[first:first + {words}] == cleared and CLEAR not in lines[first + {words}]
""")


@pytest.mark.parametrize("setup", ["grid(16, 16, 8)", "grid(16, 16, 8); double = True",
                                   "grid(64, 64, 16); lib.nh_set_jacobi_sweeps(ctx, 10)"],
                         ids=["bricks", "bricks-f64", "fixed-k"])
@pytest.mark.parametrize("after", ["", "grid(200, 160, 64)", "lib.nh_set_launch(ctx, 0, 4, 0)", "double = not double"],
                         ids=["same-plan", "other-grid", "streaming", "other-precision"])
def test_a_failed_launch_leaves_no_steps_for_the_next_call(run, setup, after):
    """The steps of a launch that failed are gone with it: the next call launches its
    own alone (the old ones point into a trajectory that has been freed)."""
    run(f"""
double = False
{setup}
for steps, failing in ((5, 1), (12, 1), (30, 2)):
    hip.host_hip_fail_cooperative(failing)
    assert forward(steps, double) == -6
    before = double
    {after or "pass"}
    hip.host_hip_reset()
    assert forward(1, double) == 0
    assert len(launches(*STEPS)) == 1, launches(*STEPS)
    double = before
    lib.nh_set_launch(ctx, 0, 0, 0)
    {setup.replace("double = True", "pass")}
""")


def test_a_failed_launch_of_an_adjoint_leaves_no_steps(run):
    run("""
grid(16, 16, 8)
assert forward(5) == 0
hip.host_hip_fail_cooperative(1)
assert adjoint(5) == -6
hip.host_hip_reset()
assert adjoint(5) == 0                       # the forward is still saved
assert len(launches(*STEPS)) == 1, launches(*STEPS)
""")


@pytest.mark.parametrize("grid,kernel", [("64, 64, 16", "jacobi_step_kernelILi"), ("40, 20, 24", "11step_kernelI")],
                         ids=["nz16", "nz24"])
def test_a_traced_fixed_k_step_runs_a_kernel_that_stamps(run, grid, kernel):
    """NH_TRACE_STEP prints the phase timings of one step: with more than 16 planes,
    where the blocked kernel has no stamps, of the streaming kernel."""
    r = run(f"""
grid({grid})
lib.nh_set_jacobi_sweeps(ctx, 6)
assert forward(3) == 0
ran = launches(*STEPS, "jacobi_step_kernel")
assert any({kernel!r} in l for l in ran) and not any("jacobi_deep" in l for l in ran), ran
""", NH_TRACE_STEP="2", NH_TRACE_RANK="0")
    assert "[nh trace] step 2" in r.stderr


@pytest.mark.parametrize("double", [False, True], ids=["f32", "f64"])
def test_bricks_hold_no_streaming_vectors(run, double):
    """The brick kernel keeps the CG state in registers: a context's memory is the
    states, the diffusivity and three banks of halo words of twice a value's size,
    and shrinks to that when a grid that streamed becomes one of bricks."""
    run(f"""
grid(64, 64, 16)
value = {8 if double else 4}
assert lib.nh_set_cg_variant(ctx, 1) == 0 and forward(6, {double}) == 0 and launches("11step_kernelI")
assert hip.host_hip_bytes() > (6 + 1 + 7) * value * cells
assert lib.nh_set_cg_variant(ctx, 2) == 0 and forward(6, {double}) == 0 and launches("brick_steps_kernel")
assert hip.host_hip_bytes() < (6 + 1 + 3 * 2) * value * cells + 2 * 64 * 256 + value * columns + 4096, hip.host_hip_bytes()
assert lib.nh_set_cg_variant(ctx, 0) == 0 and forward(6, {double}) == 0
assert lib.nh_set_cg_variant(ctx, 2) == 0 and forward(6, {double}) == 0
""")
