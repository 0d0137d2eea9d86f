"""Which kernels a plan runs, and on which device, without a GPU: libpipe.so on
a stand-in HIP runtime (fake_hip.cpp) that writes down every launch.
"""
import collections
import ctypes
import os
import re
import shutil
import subprocess
import sys

import pytest

from paper_1111_4971_amd import pipe

HERE = os.path.dirname(os.path.abspath(__file__))
HIP_INCLUDE = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(
    not (os.path.exists(pipe.LIB_PATH) and shutil.which("g++") and os.path.isdir(HIP_INCLUDE)),
    reason="needs libpipe.so, g++ and the HIP headers")

PREAMBLE = """
import ctypes, sys
sys.path[:0] = [%r, %r]
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # ahead of the runtime libpipe.so links
from paper_1111_4971_amd import pipe
from test_host_routes import *
use(fake)
"""


def use(fake):
    global _fake
    _fake = fake
    fake.fake_hip_log.restype = ctypes.c_char_p


def calls():
    """(device, kernel or "malloc") -> count since the last call."""
    c = collections.Counter()
    for line in _fake.fake_hip_log().decode().splitlines():
        dev, what, *name = line.split()
        c[int(dev), re.search(r"([a-z0-9]+_)+kernel", re.sub(r"^_ZN\d*pipe\d+", "", name[0])).group(0)
          if name else what] += 1
    _fake.fake_hip_clear()
    return c


def kernels():
    return {k for _, k in calls() if k != "malloc"}


def info(h):
    i = pipe.PlanInfo()
    pipe.check(pipe.lib().pipe_plan_info(h, ctypes.byref(i)))
    return i


def plan(shape, flags=pipe.PREC_FP32, L=(0, 0, 0), shrink=1.0):
    """A plan in a 1 x 1 pipe, on its lattice unless shrink < 1."""
    nx, ny, nz = shape
    h = ctypes.c_void_p()
    pipe.check(pipe.lib().pipe_green_plan_ex(nx, ny, nz, shrink / (nx + 1), 1.0 / (ny + 1), 0.05, 1.0, 1.0,
                                             pipe.IGF_Z | flags, 2 * nx, 2 * ny, *L, None, ctypes.byref(h)))
    return h


def solve_kernels(h, log=None):
    """The kernels of one solve; the runtime's own lines go to log."""
    buf = [ctypes.c_void_p((k + 1) << 40) for k in range(3)]       # never touched: kernels do nothing
    calls()
    pipe.check(pipe.lib().pipe_poisson_solve(h, *buf, None))
    if log is not None:
        log.append(_fake.fake_hip_log().decode())
    return kernels()


PADDED = {"z_r2c_kernel", "strided_kernel", "xprod_kernel", "z_c2r_kernel"}


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("hip") / "libfakehip.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I" + HIP_INCLUDE,
                    os.path.join(HERE, "fake_hip.cpp"), "-o", lib], check=True, timeout=120)

    def go(code, **env):
        keep = {k: v for k, v in os.environ.items() if not k.startswith("PIPE_")}
        r = subprocess.run([sys.executable, "-c", PREAMBLE % (os.path.dirname(HERE), HERE) + code, lib],
                           capture_output=True, text=True, timeout=120, env=dict(keep, **env))
        assert r.returncode == 0, r.stdout + r.stderr

    return go


def test_tuned_lengths_are_the_ones_that_run(run):
    """A lattice mesh whose lengths were tuned runs the padded passes that were timed."""
    run("""
h = plan((24, 20, 48))
assert info(h).xtile == 0 and info(h).tune_ms == -1 and "sine_kernel" in solve_kernels(h)
for flag in (pipe.AUTOTUNE, pipe.AUTOTUNE_BATCH):
    h = plan((24, 20, 48), pipe.PREC_FP32 | flag)
    assert info(h).tune_ms > 0
    assert info(h).xtile != 0 and solve_kernels(h) == PADDED
""")


def test_spectra_are_built_on_the_plans_device(run):
    """pipe_plan_spectra of a sine-mode plan, called with another device current."""
    run("""
out = ctypes.c_void_p(1 << 20)
L = pipe.lib()
for band in (None, 2):
    fake.hipSetDevice(1)
    h = plan((9, 8, 12))
    if band is not None:
        pipe.check(L.pipe_green_plan_banded(9, 8, 12, .1, 1 / 9, .05, 1., 1., 0., 0., pipe.PREC_FP32 | 1, 18, 16, 0, 0,
                                            band, 0., None, ctypes.byref(h)))
    assert info(h).xtile == 0
    fake.hipSetDevice(0)
    calls()
    if band is None:
        pipe.check(L.pipe_plan_spectra(h, out, None))
    else:
        copy = ctypes.create_string_buffer(1 << 22)
        pipe.check(L.pipe_plan_spectra(h, copy, None))
    seen = calls()
    assert seen[1, "malloc"] > 0 and {d for d, _ in seen} == {1}, seen
    now = ctypes.c_int(-1)
    fake.hipGetDevice(ctypes.byref(now))
    assert now.value == 0
""")


@pytest.mark.parametrize("schedule,padded", [(None, False), ("fixed", False), ("8,0,2048", True)])
def test_banded_plan_is_timed_against_the_plan_it_stands_for(run, schedule, padded):
    """The 3-D solve that band_speedup and PIPE_BAND_FASTEST compare with is that of the
    plan the mesh would get: padded under a forced schedule."""
    run("""
h = ctypes.c_void_p()
pipe.check(pipe.lib().pipe_green_plan_banded(24, 20, 48, 1 / 25, 1 / 21, .05, 1., 1., 0., 0., pipe.PREC_FP32 | 1, 48, 40,
                                             0, 0, 2, 0., None, ctypes.byref(h)))
assert info(h).xtile == 0
assert ("xprod_kernel" in kernels()) == %r
""" % padded, **({"PIPE_SCHEDULE": schedule} if schedule else {}))


@pytest.mark.parametrize("shape,prec,columns", [
    ((32, 32, 250), "fp32", 1), ((30, 31, 500), "fp32", 4), ((32, 32, 128), "fp64", 1), ((30, 31, 500), "fp64", 2),
    ((64, 64, 640), "fp32", 1), ((64, 64, 1000), "fp32", 4), ((64, 64, 384), "fp64", 1), ((64, 64, 500), "fp64", 2)])
def test_sine_tiles_by_depth(run, shape, prec, columns):
    """Columns a lane of the sine passes, on both sides of the limits of one and two blocks of
    depth (tiles of one column a lane: 500, 969, 256, 969; 2560, 4000, 1536, 2000)."""
    run("""
h = plan(%r, pipe.PREC_FP%s)
solve_kernels(h, last := [])
got = {int(v) for v in re.findall(r"sine_kernelI[fd]Lb[01]ELi(\\d)", last[0])}
assert got == {%d}, got
""" % (shape, prec[2:], columns))
