"""bench.py's per-kernel figures: one entry for each kernel that a plan launches, with its own
event interval and bytes, whichever way the plan solves."""
import os
import sys
from types import SimpleNamespace

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402

# band, xtile, pass bytes as pipe_plan_info reports them, and the kernels of such a plan
PLANS = {
    "padded": (-1, 8, [3, 5, 9, 5, 3], ["z_r2c", "strided", "xprod", "strided", "z_c2r"]),
    "sines": (-1, 0, [3, 5, 9, 5, 3], ["sine", "sine", "zexp", "sine", "sine"]),
    "planes": (-1, 0, [3, 5, 0, 0, 3], ["sine", "plane", "sine"]),
    "banded padded": (2, 0, [3, 9, 3, 0, 0], ["strided_pair", "xband", "strided_pair"]),
    "banded padded N=0": (0, 8, [3, 9, 3, 0, 0], ["strided_pair", "xband", "strided_pair"]),
    "banded sines": (2, 0, [3, 5, 9, 5, 3], ["sine", "sine", "zband", "sine", "sine"]),
    "banded sines, cut": (17, 0, [3, 5, 9, 5, 3], ["sine", "sine", "zconv", "sine", "sine"]),
    "banded planes": (0, 0, [3, 5, 0, 0, 3], ["sine", "plane", "sine"]),
}


@pytest.mark.parametrize("name", PLANS)
def test_every_kernel_has_its_own_figures(name):
    band, xtile, nbytes, kernels = PLANS[name]
    info = SimpleNamespace(band=band, xtile=xtile, pass_bytes=[b * 1e6 for b in nbytes])
    ms = [0.01 * (i + 1) for i in range(5)]           # the events of absent kernels take time too
    got = bench.pass_figures(info, ms)
    assert [f["kernel"].split("_kernel")[0] for f in got.values()] == kernels
    at = [i for i, b in enumerate(nbytes) if b]
    for i, f in zip(at, got.values()):
        assert f["ms"] == ms[i] and f["model_bytes"] == nbytes[i] * 1e6
        assert f["GBps"] == pytest.approx(nbytes[i] * 1e6 / (ms[i] * 1e-3) / 1e9)
        assert f["hbm_frac"] == pytest.approx(f["GBps"] / 8000)


def test_lengths_are_given_where_they_are_transformed():
    sched = dict(apad=16, zblocks=2048, xnt=0, a1pad=0, lx=256, ly=256, lz=1024)
    sine = bench.plan_lengths(SimpleNamespace(xtile=0, **sched))
    assert sine == {"solver": "sine modes", "padded_lengths": None, "schedule": None}
    padded = bench.plan_lengths(SimpleNamespace(xtile=8, **sched))
    assert padded["padded_lengths"] == [256, 256, 1024] and padded["schedule"]["x_tile"] == 8
