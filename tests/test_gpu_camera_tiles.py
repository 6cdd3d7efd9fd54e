"""The camera at the edges of its pixel tiles (16 x 4 pixels a wave): images
smaller than a tile, a tile exactly, one pixel over, rays spread so wide that a
tile's cone holds a half space, a camera close to and inside a sphere, 2 x 2
textures, and a ground seen near the horizon.  Spheres are left out of a tile
when no ray of it can hit them: images and gradients are compared with the
FP64 oracle with the tolerances of the whole-image comparison (1e-4 and 1e-3,
on pixels whose hit object is the same when every body moves by 1e-4)."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import GRAD_TOL, rel
from oracle import Oracle
from paper_1611_01652_amd import workloads as W
from test_gpu_camera import _ocam, _scene, _stable_mask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height,pitch,pos,at,texels", [
    (1, 1, 0.02, (0.3, -3.5, 1.6), (0.0, 0.0, 0.3), (32, 16)),
    (15, 3, 0.1, (0.3, -3.5, 1.6), (0.0, 0.0, 0.3), (32, 16)),
    (16, 4, 0.1, (0.3, -3.5, 1.6), (0.0, 0.0, 0.3), (2, 2)),
    (17, 5, 0.3, (0.3, -1.5, 0.6), (0.0, 0.0, 0.3), (32, 16)),     # cones wider than a half space
    (33, 9, 0.05, (0.0, -0.4, 0.5), (0.0, 0.0, 0.4), (32, 16)),    # among the spheres
    (48, 13, 0.02, (0.0, -60.0, 0.4), (0.0, 0.0, 0.3), (7, 3)),    # far away, near the horizon
])
def test_tiles_match_the_oracle(width, height, pitch, pos, at, texels):
    import torch
    from paper_1611_01652_amd.sim import Simulator
    print(f"case camera tiles {width}x{height} pitch {pitch}", flush=True)
    w, x = _scene(sizes=np.array([2, 16, 5]))
    cam = W.pinhole_camera(pos, at, focal=1.0, pitch=pitch, width=width, height=height)
    ts, tg, cell = W.synthetic_texture(*texels, 3), W.synthetic_texture(*texels, 4), 0.25
    o = Oracle(w)
    oc = _ocam(cam)
    ref, stable = _stable_mask(o, oc, ts, tg, cell, x)
    s = Simulator(w)
    xd = torch.tensor(np.ascontiguousarray(x.T), dtype=torch.float32, device="cuda")
    tsd = torch.tensor(ts, dtype=torch.float32, device="cuda")
    tgd = torch.tensor(tg, dtype=torch.float32, device="cuda")
    img = s.render(xd, cam, tsd, tgd, cell).cpu().numpy().astype(np.float64)
    assert np.abs(img - ref)[stable].max(initial=0.0) <= 1e-4
    wts = np.random.default_rng(7).normal(size=ref.shape) * stable
    g_ref = o.render_grad(oc, ts, tg, cell, wts, x=x)
    wd = torch.tensor(wts, dtype=torch.float32, device="cuda")
    g = s.render_grad(xd, cam, tsd, tgd, cell, wd).cpu().numpy().T.astype(np.float64)
    for e in range(w.n_envs):
        b = slice(w.env_body_off[e], w.env_body_off[e + 1])
        for cols in (slice(0, 3), slice(3, 12)):
            if np.abs(g_ref[b, cols]).max() == 0.0:
                assert np.abs(g[b, cols]).max() == 0.0
            else:
                assert rel(g[b, cols], g_ref[b, cols]) <= GRAD_TOL
