"""Several steps in one kernel (step graphs) against single steps: one, two and
three or four steps (the state before the last one goes to the other buffer,
which for two steps is untouched by earlier ones), with joint controls, with a
tolerance solve and a learned start, and with restitution.  Between steps the
state stays in LDS as the floats that a store and a load would carry, so both
state buffers, the carried impulses and the flags have the same bits."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_helpers import to_dev
from paper_1611_01652_amd import workloads as W

pytestmark = pytest.mark.gpu


def _model(name):
    if name == "arms":
        return W.planar_arms(n_envs=5, T=8)
    if name == "solve":
        w = W.warm_start_chains(n_envs=6, T=8, seed_salt=4, tol=1e-4, ws_w=W.wsn_init(seed_salt=2, scale=0.2))
        w.x0[:, 2] -= 0.25
        w.x0 = W.f32(w.x0)
        return w
    w = W.uneven_chains(n_envs=7, T=8, seed_salt=6)
    w.x0[:, 2] -= 0.25   # some in contact, some cut into the ground
    w.x0 = W.f32(w.x0)
    w.restitution = np.linspace(0.0, 0.8, w.n_envs).astype(np.float32)
    return w


@pytest.mark.parametrize("name", ["arms", "solve", "bouncy"])
@pytest.mark.parametrize("n", [1, 2, 3, 4])
def test_steps_in_one_kernel_equal_single_steps(name, n):
    import torch
    from paper_1611_01652_amd.sim import Simulator
    print("case steps in one kernel", name, n, flush=True)
    w = _model(name)
    s = Simulator(w)
    x0, u = to_dev(w)
    lam = torch.zeros(max(s.info.lam_size, 1), device="cuda")
    xs, le, fe = [x0.clone()], lam.clone(), None
    for k in range(n):
        xk, le, fe = s.step(xs[-1], u[k].contiguous(), le, k)
        xs.append(xk)
    buf = torch.full((2,) + tuple(x0.shape), 7.0, device="cuda")
    flags = torch.full((max(s.info.n_envs, 1),), 99, dtype=torch.int32, device="cuda")
    lg = lam.clone()
    g = s.step_graph(n, buf, u[:n].contiguous(), lg, flags=flags)
    try:
        for _ in range(3):
            buf[0].copy_(x0)
            buf[1].fill_(7.0)
            lg.copy_(lam)
            g.launch()
            torch.cuda.synchronize()
            assert torch.equal(buf[n % 2], xs[n])
            assert torch.equal(buf[(n - 1) % 2], xs[n - 1])
            assert torch.equal(lg[: le.numel()], le)
            assert torch.equal(flags, fe)
    finally:
        g.close()
    s.close()
