"""Sweeps with rows held by lanes against sweeps over the visit list.

A wave whose envs have at most one joint per pair of lanes and one placed
contact per lane keeps its constraints' rows in registers; with more contacts
than lanes it walks the visit list.  Twelve unjointed spheres in a pile place
more contacts than a team of 8 lanes has, and fewer than one of 64, so the two
widths take the two paths; chains of 2..5 bodies are run at the narrowest width
that holds their joints and at 64.  The constraint updates are the same, so every result
has the same bits, but for the friction coefficient's gradient, whose terms
are summed per lane first: rounding of a sum of n terms, bounded by
n * 2^-24 of the sum of their magnitudes; it is compared at 1e-5 relative."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import gpu_run
from paper_1611_01652_amd import workloads as W

pytestmark = pytest.mark.gpu


def _pile(n, T, store):
    rng = np.random.default_rng(1)
    pos = np.c_[rng.uniform(-0.25, 0.25, (n, 2)), rng.uniform(0.1, 0.3, n)]
    w = W.free_spheres(pos, [0.1] * n, [1.0] * n, T=T, mu=0.5)
    w.extra = {"grad_store": store}
    return w


@pytest.mark.parametrize("store", ["trajectory", "segment", "replay"])
@pytest.mark.parametrize("model", ["pile", "chains"])
def test_held_and_listed_sweeps_agree(model, store):
    def make(team):
        if model == "pile":
            w = _pile(12, 12, store)
        else:
            w = W.uneven_chains(n_envs=4, T=60, seed_salt=3, sizes=[2, 3, 4, 5])
            w.x0[:, 2] -= 0.15
            w.x0 = W.f32(w.x0)
            w.extra = {"grad_store": store}
        w.min_team = team   # (1: no wider than the envs need)
        return w

    print("case held rows", model, store, flush=True)
    a, b = gpu_run(make(1)), gpu_run(make(64))
    assert (a["flags"] == 0).all() and np.abs(a["lam_final"]).max() > 0
    for k in a:
        if k == "g_mu":
            assert np.allclose(a[k], b[k], rtol=1e-5, atol=1e-9), (a[k], b[k])
        else:
            assert np.array_equal(a[k], b[k]), k
