"""Buckets merged to the hardware queues: a few envs of many sizes give at
most one bucket per queue, every env is in exactly one, and results have the
bits of the unmerged tiling (an env's steps do not depend on its tile): one
model of all envs against a model per env.  (The friction coefficient's
gradient is summed per lane first, so it is compared at 1e-5; see the sweeps'
own comparison.)"""
from __future__ import annotations

import os

import numpy as np
import pytest

from gpu_helpers import gpu_run
from paper_1611_01652_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_merged_buckets_give_each_env_its_own_result():
    from paper_1611_01652_amd.sim import Simulator
    sizes = [2, 3, 4, 5, 6, 8, 9, 12, 14, 16, 18, 20]
    print("case merged buckets", sizes, flush=True)
    w = W.uneven_chains(n_envs=len(sizes), T=30, seed_salt=9, sizes=np.array(sizes))
    s = Simulator(w)
    queues = int(os.environ.get("GPU_MAX_HW_QUEUES", "0") or 0) or 4
    of = s.env_buckets()
    assert 1 <= len(s.teams()) <= max(queues, 1) or queues > len(sizes)
    assert of.min() == 0 and of.max() == len(s.teams()) - 1
    s.close()
    a = gpu_run(w)
    for e in (0, 3, 6, 11):
        b = gpu_run(w.subset([e]))
        sb = slice(w.env_body_off[e], w.env_body_off[e + 1])
        assert np.array_equal(a["x_final"][sb], b["x_final"])
        assert np.array_equal(a["loss"][e], b["loss"][0])
        assert np.array_equal(a["g_x0"][sb], b["g_x0"])
        assert np.allclose(a["g_mu"][e], b["g_mu"][0], rtol=1e-5, atol=1e-9)
