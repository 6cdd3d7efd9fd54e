"""Fixed-sweep rollouts of models with more tiles than the device has SIMDs
take a kernel that leaves room for two waves per SIMD: the same arithmetic, so
every env has the bits of a small model's rollout.  Arms and quadrupeds at the
edge of the rule (a tile for every SIMD, one more, and several times as many),
jointed robots with contacts, and uneven chains in several buckets."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from contact_models import lying_chains
from gpu_helpers import to_dev
from paper_1611_01652_amd import workloads as W
from paper_1611_01652_amd.sim import Simulator

pytestmark = pytest.mark.gpu

SIMDS = 4 * 256


def _rollout(w):
    s = Simulator(w)
    x0, u = to_dev(w)
    mlp = (w.extra or {}).get("mlp")
    if mlp is not None:
        u = torch.tensor(np.asarray(mlp["w"], np.float32), device="cuda")
    r = s.rollout(x0, u)
    torch.cuda.synchronize()
    out = {k: r[k].cpu().numpy() for k in ("loss", "x_final", "flags")}
    tiles = s.info.n_tiles
    s.close()
    return out, tiles


@pytest.mark.parametrize("model,envs,per_tile", [("arms", 8 * SIMDS, 8), ("arms", 8 * SIMDS + 1, 8), ("arms", 30000, 8),
                                                 ("quadruped", 3000, 2), ("lying", 6000, 2), ("chains", 6000, 0)])
def test_full_device_rollouts_have_a_small_model_s_bits(model, envs, per_tile):
    print("case full device", model, envs, flush=True)
    if model == "arms":
        w = W.planar_arms(n_envs=envs, T=6)
    elif model == "quadruped":
        w = W.quadruped(n_envs=envs, T_min=6, T_max=9, mlp_w=W.mlp_init(zero_output=False, out_scale=0.1))
    elif model == "lying":
        w = lying_chains([5] * envs, 6)
    else:
        w = W.uneven_chains(n_envs=envs, T=6, seed_salt=5)
        w.x0[:, 2] -= 0.3
        w.x0 = W.f32(w.x0)
    a, tiles = _rollout(w)
    if per_tile:
        assert tiles == (envs + per_tile - 1) // per_tile
    assert tiles > SIMDS or envs == 8 * SIMDS
    some = [0, 1, envs // 2, envs - 2, envs - 1]
    b, few = _rollout(w.subset(some))
    assert few <= SIMDS
    for i, e in enumerate(some):
        assert np.array_equal(a["loss"][e], b["loss"][i]) and a["flags"][e] == b["flags"][i]
        big = slice(w.env_body_off[e], w.env_body_off[e + 1])
        off = sum(int(w.env_body_off[k + 1] - w.env_body_off[k]) for k in some[:i])
        n = int(w.env_body_off[e + 1] - w.env_body_off[e])
        assert np.array_equal(a["x_final"][:, big], b["x_final"][:, off:off + n]), e
