"""The team widths a model accepts: powers of two from a lane for every joint
of a colour and half a lane per body, also where the model is made with wider
teams (two lanes per joint hold the joints' rows in registers, and models of
few envs take the widest that leaves every wave a CU of its own).  64
three-link arms (two joint colours, of 2 and 1 joints) take 2 to 64 lanes, and
every width gives the bits of the default.  sim_tune times the default width
first, so that with one candidate it stays."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import gpu_run, to_dev
from paper_1611_01652_amd import workloads as W
from paper_1611_01652_amd.sim import SimError, Simulator

pytestmark = pytest.mark.gpu


def test_every_width_from_the_narrowest_is_accepted_with_the_same_bits():
    w = W.planar_arms(n_envs=64, T=20)
    s = Simulator(w)
    ref = gpu_run(w, sim=s)
    default = s.teams()
    took = []
    for t in (1, 2, 4, 8, 16, 32, 64):
        print("case team width", t, flush=True)
        try:
            s.set_teams(np.full(len(default), t, np.int32))
        except SimError:
            continue
        took.append(t)
        got = gpu_run(w, sim=s)
        for k in ref:
            assert np.array_equal(got[k], ref[k]), (t, k)
    assert took == [2, 4, 8, 16, 32, 64]
    for t in (0, 3, 128):
        with pytest.raises(SimError):
            s.set_teams(np.full(len(default), t, np.int32))
    s.close()


def test_tuning_times_the_default_width_first():
    w = W.planar_arms(n_envs=64, T=20)
    s = Simulator(w)
    x0, u = to_dev(w)
    default = s.teams()
    print("case tune, arms 64 envs", default, flush=True)
    assert np.array_equal(s.tune(x0, u, max_candidates=1), default)
    s.set_teams(np.full(len(default), 4, np.int32))
    assert np.array_equal(s.tune(x0, u, max_candidates=1), default)
    assert set(s.tune(x0, u, max_candidates=7)) <= {2, 4, 8, 16, 32, 64}
    torch.cuda.synchronize()
    s.close()


def test_a_width_of_the_model_s_own_bounds_what_is_accepted():
    w = W.planar_arms(n_envs=64, T=20)
    w.min_team = 16
    s = Simulator(w)
    n = len(s.teams())
    with pytest.raises(SimError):
        s.set_teams(np.full(n, 8, np.int32))
    for t in (16, 32, 64):
        s.set_teams(np.full(n, t, np.int32))
    s.close()
