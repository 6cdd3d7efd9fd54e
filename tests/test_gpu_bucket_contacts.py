"""Merged buckets with robots on the ground: as test_gpu_buckets.py, with
chains lowered until they touch, so that carried impulses and the friction
coefficient's gradient are not zero.  Every env has the bits of a model of its
own (the friction gradient, summed per lane first, at 1e-5)."""
from __future__ import annotations

import numpy as np
import pytest

from contact_models import first_step_contacts, lying_chains
from gpu_helpers import gpu_run
from paper_1611_01652_amd.sim import Simulator

pytestmark = pytest.mark.gpu


def test_merged_buckets_in_contact_give_each_env_its_own_result():
    sizes = [2, 3, 4, 5, 6, 8, 9, 12, 14, 16, 18, 20]
    print("case merged buckets in contact", sizes, flush=True)
    w = lying_chains(sizes, 30, per_body=1)
    assert (first_step_contacts(w) > 0).all()
    s = Simulator(w)
    of = s.env_buckets()
    assert len(np.unique(of)) < len(sizes)   # some bucket holds several sizes
    s.close()
    a = gpu_run(w)
    assert np.abs(a["lam_final"]).max() > 0 and np.count_nonzero(a["g_mu"]) >= 10   # (a robot may stick)
    lam = 0
    for e in range(len(sizes)):
        b = gpu_run(w.subset([e]))
        sb = slice(w.env_body_off[e], w.env_body_off[e + 1])
        n = len(b["lam_final"])
        assert np.abs(b["lam_final"]).max() > 0
        assert np.array_equal(a["lam_final"][lam:lam + n], b["lam_final"]), e
        lam += n
        assert np.array_equal(a["x_final"][sb], b["x_final"]), e
        assert np.array_equal(a["loss"][e], b["loss"][0]), e
        assert np.array_equal(a["g_x0"][sb], b["g_x0"]), e
        assert np.allclose(a["g_mu"][e], b["g_mu"][0], rtol=1e-5, atol=1e-9), e
