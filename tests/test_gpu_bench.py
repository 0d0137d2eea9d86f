"""bench.py's figures on the GPU: fractions of the HBM peak are of the bytes the timed plans move."""
import os
import sys

import pytest

from helpers import log

pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def test_batch_fractions_are_below_the_peak():
    import torch
    assert torch.cuda.is_available()
    import bench
    from paper_1111_4971_amd import pipe, workloads
    log("bench batch leg, two replays")
    res = bench.batch_leg(pipe, torch, workloads, replays=2, warmup=1)
    fracs = {k: v for k, v in res.items() if "hbm_frac" in k}
    assert fracs and all(0 < v < 1 for v in fracs.values()), fracs
    assert res["max_member_rel_l2_fp32_vs_fp64"] < 1e-5
