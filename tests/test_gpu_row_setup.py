"""Row set-up by chunks of candidates, and sweeps to a tolerance with held rows.

The contact candidates are tested as many at a time as the team has lanes and
the placed contacts are grouped into visits chunk by chunk, so a pile of n
spheres (n ground candidates and n (n - 1) / 2 pairs) is run where its
candidates are fewer than one chunk, just fit, run over by one, and take
several, at the narrowest width and at 64 lanes.  The order in which rows take
their slots and the constraints' arithmetic do not depend on the width: every
output has the same bits.  In tolerance mode the narrow width (more contacts
than lanes) walks the visit list and the wide one holds rows in registers:
sweep and fallback counts and states are equal."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import gpu_run, to_dev
from paper_1611_01652_amd import workloads as W
from paper_1611_01652_amd.sim import Simulator

pytestmark = pytest.mark.gpu


def _pile(n, T, team):
    rng = np.random.default_rng(n)
    r = 0.25 if n < 12 else 0.35
    pos = np.c_[rng.uniform(-r, r, (n, 2)), rng.uniform(0.1, 0.3, n)]
    w = W.free_spheres(pos, [0.1] * n, [1.0] * n, T=T, mu=0.5)
    w.min_team = team
    return w


@pytest.mark.parametrize("n", [1, 2, 3, 8, 11, 12, 16])   # 1, 3, 6, 36, 66, 78, 136 candidates
def test_chunked_rows_do_not_depend_on_the_width(n):
    print("case row set-up pile", n, flush=True)
    a, b = gpu_run(_pile(n, 10, 1)), gpu_run(_pile(n, 10, 64))
    if n >= 8:   # (fewer spheres may all be in the air at the last step)
        assert np.abs(a["lam_final"]).max() > 0
    for k in a:
        if k == "g_mu":   # summed per lane first; see test_gpu_held_rows
            assert np.allclose(a[k], b[k], rtol=1e-5, atol=1e-9), (a[k], b[k])
        else:
            assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("learned", [False, True])
def test_tolerance_sweeps_held_and_listed_agree(learned):
    def run(team):
        w = W.warm_start_chains(n_envs=6, T=20, seed_salt=4, tol=1e-4, fb_tol=1e-3,
                                ws_w=W.wsn_init(seed_salt=2, scale=0.2) if learned else None)
        w.min_team = team
        s = Simulator(w)
        x0, u = to_dev(w)
        r = s.rollout_solve(x0, u)
        torch.cuda.synchronize()
        return {k: r[k].cpu().numpy() for k in ("loss", "x_final", "iters", "fallbacks", "flags")}

    print("case tolerance sweeps, learned", learned, flush=True)
    a, b = run(1), run(64)
    assert a["iters"].min() > 0
    for k in a:
        assert np.array_equal(a[k], b[k]), k
