"""Steps of models with more tiles than workgroups: several steps, and sweeps
to a tolerance, take their tiles from a queue that is cleared before every
launch, also inside a step graph; single fixed-sweep steps deal them out in
turn.  20000 arms and 24000 chains of two bodies have 2500 and 3000 tiles for
at most 2048 workgroups.  The queued steps have the bits of the dealt ones (arms:
a graph of three steps against three single steps), and of a few of the envs
as a model of their own, which has a workgroup for every tile."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_helpers import to_dev
from paper_1611_01652_amd import workloads as W
from paper_1611_01652_amd.sim import Simulator

pytestmark = pytest.mark.gpu


def _graph(s, n, x0, u, lam):
    buf = torch.zeros((2,) + tuple(x0.shape), device="cuda")
    flags = torch.zeros(s.info.n_envs, dtype=torch.int32, device="cuda")
    g = s.step_graph(n, buf, u[:n].contiguous(), lam, flags=flags)
    try:
        for _ in range(3):   # (every launch clears its queue)
            buf[0].copy_(x0)
            buf[1].fill_(7.0)
            lam.zero_()
            g.launch()
            torch.cuda.synchronize()
    finally:
        g.close()
    return buf[n % 2], buf[(n - 1) % 2], lam, flags


def test_queued_steps_equal_dealt_ones():
    print("case step queue, arms 20000", flush=True)
    w = W.planar_arms(n_envs=20000, T=3)
    s = Simulator(w)
    assert s.info.n_tiles > 2048
    x0, u = to_dev(w)
    lam = torch.zeros(s.info.lam_size, device="cuda")
    xs, le, fe = [x0], lam, None
    for k in range(3):
        xk, le, fe = s.step(xs[-1], u[k].contiguous(), le, k)
        xs.append(xk)
    x, xp, lg, flags = _graph(s, 3, x0, u, lam.clone())
    assert torch.equal(x, xs[3]) and torch.equal(xp, xs[2]) and torch.equal(lg, le) and torch.equal(flags, fe)
    s.close()


@pytest.mark.parametrize("n", [1, 2])
def test_queued_tolerance_steps_equal_a_small_model_s(n):
    print("case step queue, tolerance chains 24000, steps", n, flush=True)
    E = 24000
    w = W.uneven_chains(n_envs=E, T=2, seed_salt=7, sizes=np.full(E, 2))
    w.x0[:, 2] -= 0.4   # most in contact
    w.x0 = W.f32(w.x0)
    w.warm = 1.0
    w.extra = {"solve": dict(mode=1, tol=1e-4, max_iters=200)}
    s = Simulator(w)
    assert s.info.n_tiles > 2048
    x0, u = to_dev(w)
    x, xp, lam, flags = _graph(s, n, x0, u, torch.zeros(s.info.lam_size, device="cuda"))
    x1, _, _ = s.step(x0, u[0].contiguous(), torch.zeros(s.info.lam_size, device="cuda"), 0)
    assert torch.equal(x1, x if n == 1 else xp)
    s.close()
    some = [0, 1, 4097, 12000, 23998, 23999]
    b = w.subset(some)
    sb = Simulator(b)
    xb0, ub = to_dev(b)
    xb, _, lamb, _ = _graph(sb, n, xb0, ub, torch.zeros(sb.info.lam_size, device="cuda"))
    assert lamb.abs().max() > 0
    for i, e in enumerate(some):
        assert torch.equal(x[:, 2 * e:2 * e + 2], xb[:, 2 * i:2 * i + 2]), e
    sb.close()


def test_recurrent_units_carry_through_the_steps_of_a_graph():
    print("case step graph, recurrent controller", flush=True)
    w = W.quadruped(n_envs=24, T_min=4, T_max=4, rec=3,
                    mlp_w=W.mlp_init(W.rec_sizes(W.MLP_SIZES, 3), zero_output=False, out_scale=0.3))
    s = Simulator(w)
    x0, _ = to_dev(w)
    u = torch.tensor(np.asarray(w.extra["mlp"]["w"], np.float32), device="cuda")
    xs, le, fe = [x0], torch.zeros(s.info.lam_size, device="cuda"), None
    for k in range(4):
        xk, le, fe = s.step(xs[-1], u, le, k)
        xs.append(xk)
    buf = torch.zeros((2,) + tuple(x0.shape), device="cuda")
    lam, flags = torch.zeros_like(le), torch.zeros_like(fe)
    g = s.step_graph(4, buf, u, lam, flags=flags)
    for _ in range(3):
        buf[0].copy_(x0)
        buf[1].fill_(7.0)
        lam.zero_()
        g.launch()
        torch.cuda.synchronize()
        assert torch.equal(buf[0], xs[4]) and torch.equal(buf[1], xs[3])
        assert torch.equal(lam, le) and torch.equal(flags, fe)
    g.close()
    s.close()
