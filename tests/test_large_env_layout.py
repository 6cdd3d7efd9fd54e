"""The LDS an env needs where few of its bodies have a sphere-sphere sphere.

The row set-up keeps the spheres' world centres in LDS for envs with two
candidate pairs per body or more, and for those of up to six bodies.  The
layouts of large envs with few pairs must stay within a workgroup's 160 KB (an
env that does not fit is refused by sim_init): 460 free bodies, three of them
with a sphere-sphere sphere, need 159 KB in every reverse mode, and 164 KB if
every body had a centre.  The steps and gradients are the oracle's on both
sides of the rule."""
import numpy as np
import pytest

from oracle import Oracle
from paper_1611_01652_amd import workloads as W
from test_kernel_host_fp64 import _rel, _sizes, _store, host_fp64

LDS_BYTES = 160 * 1024


def _stride(floats):
    """Floats a workgroup reserves for an env: an odd number of float4."""
    f4 = (floats + 3) // 4
    return 4 * (f4 + (f4 % 2 == 0))


def _spheres(n, n_pair, T=1, spread=None):
    """n free spheres over the ground of which the last n_pair touch each other
    (the others pass through)."""
    rng = np.random.default_rng(n)
    r = spread or 0.12 * n ** 0.5
    pos = np.c_[rng.uniform(-r, r, (n, 2)), rng.uniform(0.1, 0.3, n)]
    w = W.free_spheres(pos, [0.1] * n, rng.uniform(0.5, 2.0, n), T=T, mu=0.5)
    w.sphere_flags = w.sphere_flags.copy()
    w.sphere_flags[: n - n_pair] &= ~W.SPHERE_PAIR
    return w


@pytest.mark.parametrize("mode", ["replay", "segment", "trajectory"])
def test_large_env_with_few_pairs_fits(mode):
    w = _store(_spheres(460, 3), mode)
    w.n_iters = 10
    w.ground = 0
    sz = _sizes(w)
    assert 4 * max(_stride(sz["fwd_floats"]), _stride(sz["adj_floats"])) <= LDS_BYTES


# pairs per body: 3/8 and 10/7 (centres formed per test), 15/7 and 10/6 (kept)
@pytest.mark.parametrize("n,n_pair", [(8, 3), (7, 5), (7, 6), (6, 5)])
def test_pairs_on_both_sides_of_the_rule_equal_the_oracle(n, n_pair):
    w = _spheres(n, n_pair, T=30, spread=0.12)
    got, o = host_fp64(w), Oracle(w)
    ref, roll = o.rollout_grad(), o.rollout()
    assert _rel(got["x_final"], roll["x_final"]) < 1e-9
    for k in ("g_x0", "g_inv_mass", "g_inv_inertia", "g_mu"):
        assert _rel(got[k], ref[k]) < 1e-9, k
