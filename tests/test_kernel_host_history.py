"""The reverse's impulse history: in LDS where a step is replayed, in the saved
working sets (global memory) where it is not.  Both hold the same records, so
the three reverse modes give the same bits: on chains with contacts, on servo
motors, with restitution, with the legged robot's controller, and on an env of
more joints than pairs of lanes in a wave (the kernel source on the host, FP64,
one-lane teams)."""
import numpy as np
import pytest

from contact_models import lying_chains
from paper_1611_01652_amd import workloads as W
from test_kernel_host_fp64 import _bouncy, _store, host_fp64


@pytest.mark.parametrize("maker", [
    lambda: lying_chains([5, 4, 7], 60),
    lambda: lying_chains([5, 6], 60, servo=True),
    lambda: lying_chains([33], 20, per_body=1),
    lambda: W.uneven_chains(n_envs=6, T=110, seed_salt=2),
    lambda: _bouncy(W.uneven_chains(n_envs=4, T=90, seed_salt=6), 0.8, seed=5),
    lambda: W.quadruped(n_envs=3, T_min=20, T_max=30, mlp_w=W.mlp_init(zero_output=False, out_scale=0.3)),
])
def test_history_in_lds_or_in_the_saved_working_sets_gives_the_same_bits(maker):
    a, b, c = (host_fp64(_store(maker(), m)) for m in ("replay", "segment", "trajectory"))
    assert np.abs(a["g_x0"]).max() > 0 and np.abs(a["g_mu"]).max() > 0
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
        np.testing.assert_array_equal(a[k], c[k], err_msg=k)
