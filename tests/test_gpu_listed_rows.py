"""Visit-list sweeps of jointed robots on the GPU against rows held by lanes.

Five-body chains lying on the ground, two ground spheres on each body, place
ten contacts and hold four joints: on teams of 8 lanes (2 lanes per joint) the
contacts do not fit the lanes and the wave walks the visit list, on 64 every row
is in registers.  The placed contacts are counted on the host.  Forward,
gradients in the three reverse modes, servo motors, and sweeps to a tolerance
with a plain and a learned start have the same bits at both widths, but for the
friction coefficient's gradient, whose terms are summed per lane first (1e-5
relative; see test_gpu_held_rows).  Chains of 40 bodies, with more joints than
pairs of lanes in the widest team, walk the list at every width: they are
compared with the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from contact_models import capacity, first_step_contacts, lying_chains
from gpu_helpers import compare_with_oracle, gpu_run, to_dev
from paper_1611_01652_amd import workloads as W
from paper_1611_01652_amd.sim import Simulator

pytestmark = pytest.mark.gpu

NARROW = 8


def _at(width, w):
    w.min_team = width if width == 64 else 1
    return w


def _teams(w):
    s = Simulator(w)
    t = s.teams().tolist()
    s.close()
    return t


def _check_contacts(w):
    n = first_step_contacts(w)
    assert (n > NARROW).all() and (n <= capacity(w)).all() and (n <= 64).all(), n


@pytest.mark.parametrize("servo", [False, True])
@pytest.mark.parametrize("store", ["trajectory", "segment", "replay"])
def test_listed_and_held_sweeps_of_jointed_robots_agree(store, servo):
    def make(width):
        # (replays keep the impulse history in LDS, where eight five-body robots
        # to a wave do not fit: four bodies with three ground spheres each)
        w = lying_chains([4, 4, 4], 30, per_body=3, servo=servo) if store == "replay" else \
            lying_chains([5, 5, 5], 30, servo=servo)
        if store == "replay":
            w.n_iters = 15
        w.extra = {"grad_store": store}
        return _at(width, w)

    print("case listed rows", store, "servo", servo, flush=True)
    _check_contacts(make(64))
    assert _teams(make(NARROW)) == [NARROW] and _teams(make(64)) == [64]
    a, b = gpu_run(make(NARROW)), gpu_run(make(64))
    assert np.abs(a["lam_final"]).max() > 0 and np.abs(a["g_mu"]).max() > 0
    for k in a:
        if k == "g_mu":
            assert np.allclose(a[k], b[k], rtol=1e-5, atol=1e-9), (a[k], b[k])
        else:
            assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("learned", [False, True])
def test_listed_and_held_tolerance_sweeps_agree(learned):
    def run(width):
        w = _at(width, lying_chains([5, 5, 5, 5], 12, tol=1e-4,
                                    net=W.wsn_init(seed_salt=2, scale=0.2) if learned else None))
        _check_contacts(w)
        s = Simulator(w)
        assert s.teams().tolist() == [NARROW if width != 64 else 64]
        x0, u = to_dev(w)
        r = s.rollout_solve(x0, u, rec_cap=4096, rec_every=1)
        torch.cuda.synchronize()
        out = {k: r[k].cpu().numpy() for k in ("loss", "x_final", "iters", "fallbacks", "flags")}
        rec = r["records"].cpu().numpy()
        s.close()
        return out, rec

    print("case listed tolerance sweeps, learned", learned, flush=True)
    (a, ra), (b, rb) = run(NARROW), run(64)
    assert a["iters"].min() > 0 and len(ra) == len(rb) > 4 * NARROW
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def test_more_joints_than_lane_pairs_equals_the_oracle():
    print("case 40-body chains", flush=True)
    w = lying_chains([40, 40], 4, per_body=1, depth=0.01)
    n = first_step_contacts(w)
    assert (n > 32).all() and (n <= capacity(w)).all()
    compare_with_oracle(w, gpu_run(w), min_state_frac=1.0)
