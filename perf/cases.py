"""What a user of this framework has it do, as cases that can be timed.

Every case is one pass through the public entry points (`Simulator`,
`WarmStartNet`): stepping, evaluating and differentiating batches of robots,
solving to a tolerance, rendering, and training the warm-start network.

    listed()             the cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  the model, handle and inputs of a case, on the GPU
    run(state)           one pass; returns its outputs whole
    work(case)           bytes and operations a pass cannot do without
    exact(case, seed)    the same outputs in 64 bits, in plain torch

A robot's topology (body counts) belongs to the case; its geometry, masses,
initial state, controls and targets come from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1611_01652_amd import workloads as W
from paper_1611_01652_amd.sim import Simulator, WarmStartNet

GRADS = ("g_x0", "g_u", "g_inv_mass", "g_inv_inertia", "g_mu", "g_damping", "g_anchor_p", "g_anchor_c")


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a policy outside the library steps a few robots: launches and latency count
        dict(name="step-arms", kind="step", model="arms", envs=64, links=3, T=1),
        # serving uneven robots: a captured sequence of steps, replayed
        dict(name="graph-chains", kind="graph", model="chains", envs=256, lo=2, hi=16, T=16),
        # the paper's ball task (section 2.1.1): restitution, one body per robot,
        # gradient descent on the initial velocities
        dict(name="train-balls", kind="train", model="balls", envs=256, T=250, how="recompute"),
        # evaluating a batch of arms on torque tapes: forward only
        dict(name="eval-arms", kind="eval", model="arms", envs=4096, links=3, T=200),
        # trajectory optimisation of the arms: the forward keeps what the reverse reads
        dict(name="train-arms", kind="train", model="arms", envs=4096, links=3, T=200, how="keep"),
        # an odd batch of longer arms on servo motors, through the checkpoints
        # (what the autograd function does)
        dict(name="train-servo-arms", kind="train", model="servo", envs=333, links=5, T=120, how="recompute"),
        # policy search for the legged robot: an MLP controller inside the step
        dict(name="train-quadrupeds", kind="train", model="quadruped", envs=512, T=60, how="keep"),
        # the benchmark's workload at a size whose working sets take a few GB
        dict(name="train-chains", kind="train", model="chains", envs=2048, lo=2, hi=32, T=120, how="keep"),
        # the same robots where memory is short: a segment's working sets at a time
        dict(name="train-chains-segments", kind="train", model="chains", envs=333, lo=2, hi=32, T=75, how="segment"),
        # solving each step to a tolerance with the learned warm start
        dict(name="solve-chains", kind="solve", model="chains", envs=512, lo=2, hi=16, T=12),
        # the differentiable camera at the paper's frame size: image and gradient
        dict(name="camera", kind="camera", model="chains", envs=512, lo=2, hi=16, T=1, width=288, height=96),
        # fitting the warm-start network: one minibatch, gradient and Adam step
        dict(name="fit-warm-start", kind="fit", model="records", records=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "graph", "balls", "eval", "arms", "servo", "quadruped", "chains", "segment", "solve",
                       "camera", "fit"])
    if kind == "step":
        return dict(kind="step", model="arms", envs=_log(rng, 1, 512), links=rng.randint(2, 6), T=1)
    if kind == "graph":
        return dict(kind="graph", model="chains", envs=_log(rng, 16, 512), lo=2, hi=rng.randint(6, 24),
                    T=rng.randint(2, 16))
    if kind == "balls":
        return dict(kind="train", model="balls", envs=_log(rng, 16, 2048), T=rng.randint(100, 250), how="recompute")
    if kind == "eval":
        return dict(kind="eval", model="arms", envs=_log(rng, 256, 4096), links=rng.randint(2, 5),
                    T=rng.randint(50, 200))
    if kind == "arms":
        return dict(kind="train", model="arms", envs=_log(rng, 256, 4096), links=rng.randint(2, 4),
                    T=rng.randint(50, 200), how=rng.choice(["keep", "recompute"]))
    if kind == "servo":
        return dict(kind="train", model="servo", envs=_log(rng, 64, 1024), links=rng.randint(2, 6),
                    T=rng.randint(40, 120), how="recompute")
    if kind == "quadruped":
        return dict(kind="train", model="quadruped", envs=_log(rng, 64, 768), T=rng.randint(20, 60),
                    how=rng.choice(["keep", "recompute"]))
    if kind == "chains":
        return dict(kind="train", model="chains", envs=_log(rng, 128, 2048), lo=2, hi=rng.randint(8, 32),
                    T=rng.randint(40, 120), how=rng.choice(["keep", "recompute"]))
    if kind == "segment":
        return dict(kind="train", model="chains", envs=_log(rng, 64, 512), lo=2, hi=rng.randint(8, 32),
                    T=rng.randint(30, 75), how="segment")
    if kind == "solve":
        return dict(kind="solve", model="chains", envs=_log(rng, 64, 512), lo=2, hi=rng.randint(6, 16),
                    T=rng.randint(4, 12))
    if kind == "camera":
        return dict(kind="camera", model="chains", envs=_log(rng, 16, 512), lo=2, hi=rng.randint(4, 16), T=1,
                    width=rng.randint(64, 288), height=rng.randint(48, 96))
    return dict(kind="fit", model="records", records=_log(rng, 100, 65536))


# ------------------------------------------------------------------ inputs
def _bodies(case):
    """Body counts of the case's chains: the uneven-chain distribution."""
    rng = np.random.default_rng([case["envs"], case["lo"], case["hi"]])
    return W.chain_sizes(case["envs"], rng, lo=case["lo"], hi=case["hi"])


def _workload(case, seed):
    T = case["T"]
    if case["model"] == "arms":
        w = W.planar_arms(n_envs=case["envs"], T=T, seed_salt=seed, n_links=case["links"])
    elif case["model"] == "servo":
        base = W.planar_arms(n_envs=case["envs"], T=T, seed_salt=seed, n_links=case["links"])
        base.gravity = (0.0, -9.81, 0.0)
        w = W.with_servos(base, gain=10.0, torque=50.0, vmax=3.0,
                          targets=W.servo_targets(T, base.n_joints, seed_salt=seed, amp=0.8, hold=30))
    elif case["model"] == "balls":
        w = W.paper_ball_throws(n_envs=case["envs"], T=T, seed_salt=seed)
    elif case["model"] == "quadruped":
        w = W.quadruped(n_envs=case["envs"], T_min=T, T_max=T, seed_salt=seed,
                        mlp_w=W.mlp_init(seed_salt=seed, zero_output=False, out_scale=0.1))
    else:
        w = W.uneven_chains(n_envs=case["envs"], T=T, seed_salt=seed, sizes=_bodies(case))
        if case["kind"] == "solve":
            # a network as training leaves it: small corrections to the carried impulses
            net = W.wsn_init(seed_salt=seed)
            net[-195:] *= 0.02
            w.warm = 1.0
            w.extra = {"solve": dict(mode=1, tol=1e-4, max_iters=1000), "ws": dict(w=net, fb_iters=5, fb_tol=1e-3)}
        if case["kind"] == "camera":
            # part of the way down, so that the camera sees robots over and on the ground
            w.x0[:, 2] -= np.repeat(np.random.default_rng(seed).uniform(0.0, 0.2, w.n_envs), np.diff(w.env_body_off))
            w.x0 = W.f32(w.x0)
    if case.get("how") == "segment":
        w.ckpt_every = 25
        w.extra = dict(w.extra or {}, grad_store="segment")
    elif case["kind"] == "train":
        w.extra = dict(w.extra or {}, grad_store="trajectory")
    return w


def _scene(case, seed):
    wd, hg = case["width"], case["height"]
    cam = W.pinhole_camera((0.3, -3.5, 1.6), (0.0, 0.0, 0.3), focal=1.0, pitch=1.6 / wd, width=wd, height=hg)
    rng = np.random.default_rng([seed, 7])
    # adjoint of an image, as a loss on the image leaves it
    weights = rng.standard_normal((case["envs"], hg, wd), dtype=np.float32)
    return cam, W.synthetic_texture(64, 32, seed), W.synthetic_texture(64, 64, seed + 1), 0.25, weights


def _records(case, seed):
    """Contact records as the solver writes them (include/sim.h): features,
    converged impulses over their effective masses, in m/s."""
    n = case["records"]
    rng = np.random.default_rng([seed, 9])
    r = np.zeros((n, 16), np.float32)
    r[:, 0] = rng.uniform(-2, 10, n)
    r[:, 1:4] = rng.normal(0, 0.5, (n, 3))
    r[:, 4] = np.abs(rng.normal(0, 0.1, n))
    r[:, 5:7] = rng.normal(0, 0.05, (n, 2))
    r[:, 7] = np.maximum(r[:, 4] - 0.3 * r[:, 1], 0)
    r[:, 8:10] = 0.5 * r[:, 5:7] - 0.1 * r[:, 2:4]
    r[:, 10:12] = 1.0
    return r, W.wsn_init(seed_salt=seed)


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")


def _controls(w):
    mlp = (w.extra or {}).get("mlp")
    if mlp is not None:
        return mlp["w"]
    return w.u if w.u.size else np.zeros((w.T_max, 1))


def prepare(case, seed):
    s = {"case": case}
    if case["kind"] == "fit":
        rec, w0 = _records(case, seed)
        s["net"], s["rec"] = WarmStartNet(w0), _dev(rec)
        return s
    w = _workload(case, seed)
    sim = s["sim"] = Simulator(w)
    s["x0"] = _dev(w.x0.T)
    s["u"] = _dev(_controls(w))
    if case["kind"] == "train":
        s["dloss"] = torch.ones(w.n_envs, device="cuda")
        s["ws"] = sim.workspace()
    elif case["kind"] == "step":
        s["lam"] = torch.zeros(sim.info.lam_size, device="cuda")
    elif case["kind"] == "graph":
        s["x"] = torch.empty((2,) + tuple(s["x0"].shape), device="cuda")
        s["lam"] = torch.zeros(sim.info.lam_size, device="cuda")
        s["graph"] = sim.step_graph(case["T"], s["x"], s["u"], s["lam"])
    elif case["kind"] == "camera":
        s["cam"], ts, tg, s["cell"], wt = _scene(case, seed)
        s["ts"], s["tg"], s["wt"] = _dev(ts), _dev(tg), _dev(wt)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "fit":
        net = s["net"]
        loss, grad = net.loss_grad(s["rec"], huber=0.05, relative=True)
        net.adam(1e-3)
        return dict(loss=loss, grad=grad, w=net.w, m=net.m, v=net.v)
    sim = s["sim"]
    if kind == "step":
        x, lam, flags = sim.step(s["x0"], s["u"][0], s["lam"])
        return dict(x=x, lam=lam, flags=flags)
    if kind == "graph":
        s["x"][0].copy_(s["x0"])
        s["lam"].zero_()
        s["graph"].launch()
        return dict(x=s["x"][s["case"]["T"] % 2], lam=s["lam"])
    if kind == "eval":
        r = sim.rollout(s["x0"], s["u"], want_ckpt=False)
        return dict(loss=r["loss"], x=r["x_final"], flags=r["flags"])
    if kind == "solve":
        r = sim.rollout_solve(s["x0"], s["u"])
        return dict(loss=r["loss"], x=r["x_final"], iters=r["iters"], fallbacks=r["fallbacks"], flags=r["flags"])
    if kind == "camera":
        img = sim.render(s["x0"], s["cam"], s["ts"], s["tg"], s["cell"])
        g = sim.render_grad(s["x0"], s["cam"], s["ts"], s["tg"], s["cell"], s["wt"])
        return dict(image=img, g_x=g)
    if s["case"]["how"] == "keep":
        r = sim.rollout(s["x0"], s["u"], want_ckpt=False, keep=s["ws"])
        g = sim.rollout_grad(s["x0"], s["u"], None, s["dloss"], kept=s["ws"])
    else:
        r = sim.rollout(s["x0"], s["u"])
        g = sim.rollout_grad(s["x0"], s["u"], r["ckpt"], s["dloss"], workspace=s["ws"])
    out = {k: g[k] for k in GRADS}
    out.update(loss=r["loss"], x=r["x_final"], flags=r["flags"], grad_flags=g["flags"])
    return out


# ------------------------------------------------------------------ work
def _counts(case):
    """(bodies, joints, spheres, controls per step) of a case's batch."""
    E, m = case["envs"], case["model"]
    if m in ("arms", "servo"):
        n = E * case["links"]
        return n, n, 0, n
    if m == "balls":
        return E, 0, E, 0
    if m == "quadruped":
        return 9 * E, 8 * E, 8 * E, 0
    B = int(_bodies(case).sum())
    return B, B - E, B, B - E


def work(case):
    """Inputs read once and outputs written once; operations of the step as
    it is defined (20 sweeps, five rows of 46 operations per hinge, three per
    contact with about half of the spheres in contact), the reverse at 2.7
    operations per forward one beyond the forward itself."""
    if case["kind"] == "fit":
        n, p = case["records"], W.WSN_PARAMS
        return {"bytes": 4.0 * (10 * n + 3 * p + 4 * p) + 2 * p, "flops": 6.0 * p * n}
    B, J, S, nu = _counts(case)
    E, T = case["envs"], case["T"]
    if case["kind"] == "camera":
        pix = float(case["width"] * case["height"])
        return {"bytes": 8.0 * E * pix + 4 * 36 * B, "flops": 2 * pix * (27.0 * E + 45.0 * S)}
    rows = 6 if case["model"] == "servo" else 5
    step = 300.0 * B + J * (800 + 20 * 46.0 * rows) + 0.5 * S * (300 + 20 * 150.0)
    if case["model"] == "quadruped":
        step += 2.0 * E * W.mlp_param_count(W.MLP_SIZES)
    words = 2 * 18.0 * B + nu * T
    flops = step * T
    if case["kind"] == "train":
        words += 18.0 * B + nu * T + 4 * B + 7 * J + 2 * E
        flops *= 3.7
    elif case["kind"] in ("step", "graph"):
        words += 2.0 * (rows * J + 4 * S)
    return {"bytes": 4.0 * words, "flops": flops}


# ------------------------------------------------------------------ 64 bits
def _dot(a, b):
    return (a * b).sum(-1)


def _mv(R, v):
    return (R @ v.unsqueeze(-1)).squeeze(-1)


def _colours(w):
    """The visits of a sweep, first to last, as (kind, rows) over all robots
    at once: hinges by greedy colour in index order, ground spheres by their
    rank among their body's, sphere pairs by round-robin rounds."""
    joints, ground, pairs = {}, {}, {}
    for e in range(w.n_envs):
        b0, b1 = int(w.env_body_off[e]), int(w.env_body_off[e + 1])
        used, linked = {}, set()
        for j in range(int(w.env_joint_off[e]), int(w.env_joint_off[e + 1])):
            p, c = int(w.joint_parent[j]), int(w.joint_child[j])
            taken = used.setdefault(c, set()) | (used.setdefault(p, set()) if p >= 0 else set())
            col = next(k for k in range(len(taken) + 1) if k not in taken)
            used[c].add(col)
            if p >= 0:
                used[p].add(col)
            linked.add((min(p, c), max(p, c)))
            joints.setdefault(col, []).append(j)
        rank, ball = {}, {}
        for k in range(int(w.env_sphere_off[e]), int(w.env_sphere_off[e + 1])):
            b = int(w.sphere_body[k])
            if w.ground and w.sphere_flags[k] & 1:
                ground.setdefault(rank.get(b, 0), []).append(k)
                rank[b] = rank.get(b, 0) + 1
            if w.sphere_flags[k] & 2:
                ball[b] = k
        n = b1 - b0 + (b1 - b0) % 2
        for k in range(n - 1):
            for i in range(n // 2):
                x, y = (k, n - 1) if i == 0 else ((k + i) % (n - 1), (k - i) % (n - 1))
                x, y = b0 + min(x, y), b0 + max(x, y)
                if x in ball and y in ball and (x, y) not in linked:
                    pairs.setdefault(k, []).append((ball[x], ball[y]))
    return joints, ground, pairs


class _Reference:
    """The batch's step x^{t+1} = f(x^t, u^t) in 64 bits over all robots at
    once, differentiable by torch."""

    def __init__(self, w, device):
        t = lambda a, k=torch.float64: torch.tensor(np.asarray(a), device=device).to(k)  # noqa: E731
        self.w, self.t, self.B = w, t, w.n_bodies
        f = lambda v: float(np.float32(v))  # noqa: E731
        self.dt, self.beta, self.spec, self.warm = f(w.dt), f(w.beta), f(w.spec_margin), f(w.warm)
        self.g = t([f(v) for v in w.gravity])
        self.env = t(np.repeat(np.arange(w.n_envs), np.diff(w.env_body_off)), torch.long)
        self.a = t(np.where(w.joint_parent < 0, self.B, w.joint_parent), torch.long)   # the world is body B
        self.b = t(w.joint_child, torch.long)
        self.par = dict(inv_mass=t(w.inv_mass), inv_inertia=t(w.inv_inertia), mu=t(w.mu), damping=t(w.damping),
                        anchor_p=t(w.anchor_p), anchor_c=t(w.anchor_c))
        self.axis_p, self.axis_c, self.perp_p, self.perp_c = (t(v) for v in (w.axis_p, w.axis_c, w.perp_p, w.perp_c))
        self.rest = t(np.zeros(w.n_envs) if w.restitution is None else w.restitution)
        self.servo = None if w.servo_gain is None else (t(w.servo_gain), t(w.servo_torque), t(w.servo_vmax))
        self.sph_b, self.sph_o, self.sph_r = t(w.sphere_body, torch.long), t(w.sphere_offset), t(w.sphere_radius)
        joints, ground, pairs = _colours(w)
        self.jcol = [t(v, torch.long) for _, v in sorted(joints.items())]
        # contact candidates: spheres (i, k), i = -1 the ground, each with its visit
        ci = [(-1, k, c) for c, v in sorted(ground.items()) for k in v]
        ci += [(i, k, len(ground) + c) for c, v in sorted(pairs.items()) for i, k in v]
        self.cand = t(np.array(ci, np.int64).reshape(-1, 3), torch.long)
        mlp = (w.extra or {}).get("mlp")
        self.clock = None if mlp is None else f(mlp["clock_hz"])

    def start(self):
        z = lambda *n: torch.zeros(n, dtype=torch.float64, device=self.g.device)  # noqa: E731
        return z(len(self.a), 5 if self.servo is None else 6), z(len(self.cand), 4)

    def _controller(self, W_, R, v6, t):
        n_in, h1, h2, n_out = W.MLP_SIZES
        E = self.w.n_envs
        na, ua = _mv(R[self.a], self.axis_p), _mv(R[self.a], self.perp_p)
        ub = _mv(R[self.b], self.perp_c)
        th = torch.atan2(_dot(torch.linalg.cross(ua, ub), na), _dot(ua, ub)).view(E, -1)
        rate = _dot(v6[self.b, 3:] - v6[self.a, 3:], na).view(E, -1)
        ph = 2 * math.pi * self.clock * t * self.dt
        ck = torch.tensor([math.sin(ph), math.cos(ph)], dtype=torch.float64, device=W_.device)
        s, o = torch.cat([th, rate, ck.expand(E, 2)], 1), 0
        for a, b, last in ((n_in, h1, 0), (h1, h2, 0), (h2, n_out, 1)):
            s = s @ W_[o:o + a * b].view(b, a).T + W_[o + a * b:o + a * b + b]
            s, o = (s if last else torch.tanh(s)), o + a * b + b
        return s.reshape(-1)

    def _apply(self, V, idx, dv):
        return V.index_add(0, idx, dv)

    def _contact_rows(self, p, R, V, I, im, lam_c):
        """The active contacts of the step, by visit."""
        one = torch.ones_like
        i, k = self.cand[:, 0], self.cand[:, 1]
        bb, gnd = self.sph_b[k], i < 0
        ba = torch.where(gnd, torch.full_like(bb, self.B), self.sph_b[i.clamp(min=0)])
        with torch.no_grad():
            cen = p[self.sph_b] + _mv(R[self.sph_b], self.sph_o)
            d = cen[k] - cen[i.clamp(min=0)]
            gap = torch.where(gnd, cen[k, 2], _dot(d, d).sqrt() - self.sph_r[i.clamp(min=0)]) - self.sph_r[k]
            on = torch.nonzero(gap < self.spec).view(-1)
        i, k, ba, bb, gnd = i[on], k[on], ba[on], bb[on], gnd[on].unsqueeze(-1)
        if not len(on):
            return on, []
        ez, ex, ey = (self.t([[0., 0., 1.]]), self.t([[1., 0., 0.]]), self.t([[0., 1., 0.]]))
        cb = p[bb] + _mv(R[bb], self.sph_o[k])
        ca = p[ba] + _mv(R[ba], self.sph_o[i.clamp(min=0)])
        d = torch.where(gnd, ez, cb - ca)
        L = _dot(d, d).sqrt().unsqueeze(-1)
        n = torch.where(gnd, ez, d / L)
        rk, ri = self.sph_r[k].unsqueeze(-1), self.sph_r[i.clamp(min=0)].unsqueeze(-1)
        gap = torch.where(gnd, cb[:, 2:], L - ri) - rk
        ra, rb = ca + ri * n - p[ba], cb - rk * n - p[bb]
        e = torch.where(n[:, 2:].abs() < 0.9, ez, ex)
        wv = torch.linalg.cross(n, e)
        t1 = torch.where(gnd, ex, wv / _dot(wv, wv).sqrt().unsqueeze(-1))
        t2 = torch.where(gnd, ey, torch.linalg.cross(n, t1))
        dirs = torch.stack([n, t1, t2], 1)
        off = (~gnd).double().unsqueeze(-1)
        Jb = torch.cat([dirs, torch.linalg.cross(rb.unsqueeze(1).expand_as(dirs), dirs)], -1)
        Ja = torch.cat([-dirs, torch.linalg.cross(dirs, ra.unsqueeze(1).expand_as(dirs))], -1) * off
        Wa, Wb = self._minv(Ja, ba, I, im), self._minv(Jb, bb, I, im)
        K = _dot(Ja, Wa) + _dot(Jb, Wb)
        gap = gap.squeeze(-1)
        bias = torch.where(gap > 0, gap, self.beta * gap) / self.dt
        er = self.rest[self.env[bb]]
        vn = _dot(Jb[:, 0], V[bb]) + _dot(Ja[:, 0], V[ba])
        hit = (er > 0) & (vn < -float(np.float32(self.w.rest_threshold))) & (vn * self.dt + gap < 0) & (er * vn < bias)
        bias = torch.where(hit, er * vn, bias)
        lc = self.warm * lam_c[on]
        l0 = torch.stack([lc[:, 0], _dot(t1, lc[:, 1:]), _dot(t2, lc[:, 1:])], 1)
        mu = self.mu[self.env[bb]]
        col = self.cand[on, 2]
        vis = []
        for c in torch.unique(col).tolist():
            s = torch.nonzero(col == c).view(-1)
            vis.append(dict(s=s, a=ba[s], b=bb[s], Ja=Ja[s], Jb=Jb[s], Wa=Wa[s], Wb=Wb[s], mn=1 / K[s, 0],
                            mt=2 / (K[s, 1] + K[s, 2]), bias=bias[s], mu=mu[s], lam=l0[s], t1=t1[s], t2=t2[s]))
        return on, vis

    def _minv(self, J, body, I, im):
        return torch.cat([J[..., :3] * im[body].view(-1, 1, 1), J[..., 3:] @ I[body]], -1)   # (I symmetric)

    def step(self, x, u, lam, t, par):
        """x [B, 18] -> x' [B, 18]; u the controls of the step, or the controller's weights."""
        lam_j, lam_c = lam
        z1 = torch.zeros(1, 18, dtype=torch.float64, device=x.device)
        xw = torch.cat([x, z1])
        p, R, V = xw[:, :3], xw[:, 3:12].view(-1, 3, 3), xw[:, 12:]
        R = torch.cat([R[:-1], torch.eye(3, dtype=torch.float64, device=x.device).unsqueeze(0)])
        im = torch.cat([par["inv_mass"], z1[0, :1]])
        iI = torch.cat([par["inv_inertia"], z1[:, :3]])
        self.mu = par["mu"]
        I = (R * iI.unsqueeze(1)) @ R.transpose(1, 2)
        a, b = self.a, self.b
        if self.clock is not None:
            u = self._controller(u, R, V, t)
        dv = torch.zeros_like(V)
        world = (a < self.B).unsqueeze(-1)
        if len(a):
            na = _mv(R[a], self.axis_p)
            tau = (0.0 if self.servo else u) - par["damping"] * _dot(V[b, 3:] - V[a, 3:], na)
            tq = torch.zeros_like(p).index_add(0, b, tau.unsqueeze(-1) * na).index_add(0, a, -tau.unsqueeze(-1) * na)
            dv = torch.cat([dv[:, :3], self.dt * _mv(I, tq)], -1)
        live = (torch.arange(self.B + 1, device=x.device) < self.B).double().unsqueeze(-1)
        V = (V + dv + torch.cat([self.dt * self.g, torch.zeros_like(self.g)])) * live
        # hinge rows: the point (world axes), two directions normal to the axis, a servo's motor row
        if len(a):
            rb, ra = _mv(R[b], par["anchor_c"]), _mv(R[a], par["anchor_p"])
            err = p[b] + rb - p[a] - ra
            ua = _mv(R[a], self.perp_p)
            t2 = _mv(R[a], torch.linalg.cross(self.axis_p, self.perp_p))
            ax = torch.linalg.cross(na, _mv(R[b], self.axis_c))
            eye = torch.eye(3, dtype=torch.float64, device=x.device).expand(len(a), 3, 3)
            ang = [ua, t2] + ([na] if self.servo else [])
            kb = self.beta / self.dt
            bias = torch.cat([kb * err, kb * torch.stack([_dot(ua, ax), _dot(t2, ax)], 1)], 1)
            if self.servo:
                gain, tmax, vmax = self.servo
                ub = _mv(R[b], self.perp_c)
                th = torch.atan2(_dot(torch.linalg.cross(ua, ub), na), _dot(ua, ub))
                bias = torch.cat([bias, -torch.clamp(gain * (u - th), -vmax, vmax).unsqueeze(-1)], 1)
            zero = torch.zeros_like(torch.stack(ang, 1))
            Jb = torch.cat([torch.cat([eye, torch.linalg.cross(rb.unsqueeze(1).expand(-1, 3, 3), eye)], -1),
                            torch.cat([zero, torch.stack(ang, 1)], -1)], 1)
            Ja = torch.cat([torch.cat([-eye, torch.linalg.cross(eye, ra.unsqueeze(1).expand(-1, 3, 3))], -1),
                            torch.cat([zero, -torch.stack(ang, 1)], -1)], 1) * world.unsqueeze(-1)
            Wb, Wa = self._minv(Jb, b, I, im), self._minv(Ja, a, I, im)
            K = Jb @ Wb.transpose(1, 2) + Ja @ Wa.transpose(1, 2)
            m = 1 / torch.diagonal(K, dim1=1, dim2=2)
            # five unbounded rows one after another: d = -(diag(1/m) + strict lower K)^-1 s
            low = torch.linalg.inv(torch.tril(K[:, :5, :5]))
            lj = [self.warm * lam_j[c] for c in self.jcol]
        on, vis = self._contact_rows(p, R, V, I, im, lam_c)
        if len(a):
            for c, l in zip(self.jcol, lj):
                V = self._apply(V, b[c], (Wb[c] * l.unsqueeze(-1)).sum(1))
                V = self._apply(V, a[c], (Wa[c] * l.unsqueeze(-1)).sum(1))
            hinges = [(c, a[c], b[c], Ja[c], Jb[c], Wa[c], Wb[c], low[c], bias[c], m[c]) for c in self.jcol]
        else:
            hinges, lj = [], []
        for v in vis:
            V = self._apply(V, v["b"], (v["Wb"] * v["lam"].unsqueeze(-1)).sum(1))
            V = self._apply(V, v["a"], (v["Wa"] * v["lam"].unsqueeze(-1)).sum(1))
        for _ in range(self.w.n_iters):
            for q, (c, ca, cb, ja, jb, wa, wb, lw, bi, mm) in enumerate(hinges):
                va, vb = V[ca], V[cb]
                s = (jb[:, :5] @ vb.unsqueeze(-1) + ja[:, :5] @ va.unsqueeze(-1)).squeeze(-1) + bi[:, :5]
                d = -_mv(lw, s)
                dva, dvb = (wa[:, :5] * d.unsqueeze(-1)).sum(1), (wb[:, :5] * d.unsqueeze(-1)).sum(1)
                if self.servo:
                    s6 = _dot(jb[:, 5], vb + dvb) + _dot(ja[:, 5], va + dva) + bi[:, 5]
                    hi = self.servo[1][c] * self.dt
                    l6 = lj[q][:, 5] - mm[:, 5] * s6
                    d6 = torch.minimum(torch.maximum(l6, -hi), hi) - lj[q][:, 5]
                    dva, dvb = dva + wa[:, 5] * d6.unsqueeze(-1), dvb + wb[:, 5] * d6.unsqueeze(-1)
                    d = torch.cat([d, d6.unsqueeze(-1)], 1)
                V = self._apply(self._apply(V, cb, dvb), ca, dva)
                lj[q] = lj[q] + d
            for v in vis:
                va, vb, l = V[v["a"]], V[v["b"]], v["lam"]
                s = _dot(v["Jb"][:, 0], vb) + _dot(v["Ja"][:, 0], va) + v["bias"]
                ln = torch.clamp(l[:, 0] - v["mn"] * s, min=0.0)
                d0 = (ln - l[:, 0]).unsqueeze(-1)
                va, vb = va + v["Wa"][:, 0] * d0, vb + v["Wb"][:, 0] * d0
                lt = l[:, 1:] - v["mt"].unsqueeze(-1) * (_dot(v["Jb"][:, 1:], vb.unsqueeze(1)) +
                                                         _dot(v["Ja"][:, 1:], va.unsqueeze(1)))
                q2, rho = _dot(lt, lt), v["mu"] * ln
                out = q2 > rho * rho
                sc = torch.where(out, rho / torch.where(out, q2, torch.ones_like(q2)).sqrt(), torch.ones_like(q2))
                lt = sc.unsqueeze(-1) * lt
                v["lam"] = torch.cat([ln.unsqueeze(-1), lt], 1)
                dl = (v["lam"] - l).unsqueeze(-1)
                V = self._apply(V, v["b"], (v["Wb"] * dl).sum(1))
                V = self._apply(V, v["a"], (v["Wa"] * dl).sum(1))
        lam_j2, lam_c2 = torch.zeros_like(lam_j), torch.zeros_like(lam_c)
        for c, l in zip(self.jcol, lj):
            lam_j2 = lam_j2.index_add(0, c, l)
        for v in vis:
            l = v["lam"]
            lam_c2 = lam_c2.index_add(0, on[v["s"]], torch.cat([l[:, :1], l[:, 1:2] * v["t1"] + l[:, 2:] * v["t2"]], 1))
        V, R = V[:-1], R[:-1]
        w3 = V[:, 3:]
        A = R + self.dt * torch.linalg.cross(w3.unsqueeze(-1).expand_as(R), R, dim=1)
        R = 1.5 * A - 0.5 * A @ (A.transpose(1, 2) @ A)
        return torch.cat([p[:-1] + self.dt * V[:, :3], R.reshape(-1, 9), V], 1), (lam_j2, lam_c2)

    def loss(self, x, t):
        """Every robot's loss term of the state x after step t (from 1)."""
        w = self.w
        q = x[self.t(w.loss_body, torch.long)]
        mask = self.t([(w.loss_mask >> k) & 1 for k in range(3)])
        d = (q[:, :3] - self.t(w.target)) * mask
        if w.loss_kind == W.LOSS_MEAN_DIST:
            return _dot(d, d).sqrt() / w.T_max
        if t != w.T_max:
            return None
        if w.loss_kind == W.LOSS_FINAL_SQDIST:
            return _dot(d, d)
        if w.loss_kind == W.LOSS_FINAL_STATE:
            return _dot(d, d) + _dot(q[:, 12:], q[:, 12:])
        return -(q[:, 0] - self.t(w.x0)[self.t(w.loss_body, torch.long), 0]) / (w.T_max * self.dt)


def _exact_rollout(case, seed):
    w = _workload(case, seed)
    ref = _Reference(w, "cuda" if torch.cuda.is_available() else "cpu")
    t = ref.t
    U = t(_controls(w))
    at = (lambda k: U) if ref.clock is not None else (lambda k: U[k, :w.n_joints])
    x, lam, loss, kept = t(w.x0), ref.start(), torch.zeros(w.n_envs, dtype=torch.float64, device=ref.g.device), []
    with torch.no_grad():
        for k in range(w.T_max):
            kept.append((x, lam))
            x, lam = ref.step(x, at(k), lam, k, ref.par)
            term = ref.loss(x, k + 1)
            loss = loss if term is None else loss + term
    soa = lambda v: v.T.contiguous().cpu()  # noqa: E731
    if case["kind"] in ("step", "graph"):
        return dict(x=soa(x), lam=None, flags=None)
    if case["kind"] == "eval":
        return dict(loss=loss.cpu(), x=soa(x), flags=None)
    # back through the steps, one at a time
    gx, gl = torch.zeros_like(x), tuple(torch.zeros_like(v) for v in lam)
    gu = torch.zeros_like(U)
    gp = {k: torch.zeros_like(v) for k, v in ref.par.items()}
    for k in reversed(range(w.T_max)):
        xs, ls = kept[k][0].detach().requires_grad_(), tuple(v.detach().requires_grad_() for v in kept[k][1])
        uk = at(k).detach().requires_grad_()
        par = {n: v.detach().requires_grad_() for n, v in ref.par.items()}
        x1, l1 = ref.step(xs, uk, ls, k, par)
        term = ref.loss(x1, k + 1)
        total = (x1 * gx).sum() + sum((v * g).sum() for v, g in zip(l1, gl)) + (0 if term is None else term.sum())
        leaves = [xs, *ls, uk, *par.values()]
        got = [torch.zeros_like(v) if g is None else g
               for v, g in zip(leaves, torch.autograd.grad(total, leaves, allow_unused=True))]
        gx, gl = got[0], tuple(got[1:3])
        if ref.clock is not None:
            gu += got[3]
        else:
            gu[k, :w.n_joints] = got[3]
        for n, g in zip(par, got[4:]):
            gp[n] += g
    if w.loss_kind == W.LOSS_NEG_MEAN_VELX:
        gx[t(w.loss_body, torch.long), 0] += 1 / (w.T_max * ref.dt)
    out = {"g_" + k: v.cpu() for k, v in gp.items()}
    out.update(loss=loss.cpu(), x=soa(x), g_x0=soa(gx), flags=None, grad_flags=None)
    out["g_u"] = (gu if ref.clock is not None else gu[:, :w.n_joints]).cpu() if w.n_joints else None
    return out


def _bilinear(T, u, v):
    ny, nx = T.shape
    fu, fv = u - u.detach().floor(), v - v.detach().floor()
    a, b = u.detach().floor().long(), v.detach().floor().long()
    s = lambda j, i: T[(b + j) % ny, (a + i) % nx]  # noqa: E731
    return (1 - fu) * (1 - fv) * s(0, 0) + fu * (1 - fv) * s(0, 1) + (1 - fu) * fv * s(1, 0) + fu * fv * s(1, 1)


def _exact_camera(case, seed):
    w = _workload(case, seed)
    cam, ts, tg, cell, wt = _scene(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float64, device=dev)  # noqa: E731
    ts, tg, wt = t(np.float32(ts)), t(np.float32(tg)), t(wt)
    H, Wd = case["height"], case["width"]
    u = (torch.arange(Wd, dtype=torch.float64, device=dev) + 0.5 - 0.5 * Wd) * cam["pitch"]
    v = (0.5 * H - torch.arange(H, dtype=torch.float64, device=dev) - 0.5) * cam["pitch"]
    ax, C = t(cam["axes"]), t(cam["pos"])
    d = (cam["focal"] * ax[2] + u.view(1, -1, 1) * ax[0] + v.view(-1, 1, 1) * ax[1]).view(-1, 3)
    sg = torch.where(d[:, 2] != 0, -C[2] / d[:, 2], torch.full_like(d[:, 2], -1.0))
    hit_g = sg >= 1.0
    far = torch.where(hit_g, sg, torch.full_like(sg, math.inf))
    hg = C + torch.where(hit_g, sg, torch.ones_like(sg)).unsqueeze(-1) * d
    colour_g = torch.where(hit_g, _bilinear(tg, hg[:, 0] / cell, hg[:, 1] / cell), torch.zeros_like(sg))
    images, grads = [], []
    A = _dot(d, d).unsqueeze(-1)
    for e in range(w.n_envs):
        b0, b1 = int(w.env_body_off[e]), int(w.env_body_off[e + 1])
        k0, k1 = int(w.env_sphere_off[e]), int(w.env_sphere_off[e + 1])
        x = t(w.x0[b0:b1, :12]).requires_grad_()
        body = torch.tensor(w.sphere_body[k0:k1] - b0, device=dev).long()
        R = x[:, 3:].view(-1, 3, 3)[body]
        cen, r = x[body, :3] + _mv(R, t(w.sphere_offset[k0:k1])), t(w.sphere_radius[k0:k1])
        m = C - cen
        with torch.no_grad():
            bq = d @ m.T
            disc = bq * bq - A * (_dot(m, m) - r * r)
            root = disc.clamp(min=0).sqrt()
            s = torch.where((-bq - root) / A >= 1, (-bq - root) / A, (-bq + root) / A)
            s = torch.where((disc >= 0) & (s >= 1), s, torch.full_like(s, math.inf))
            best, k = s.min(1)
            px = torch.nonzero(best < far).view(-1)
            k = k[px]
        dd, mm, rr = d[px], m[k], r[k]
        Aq, Bq = _dot(dd, dd), _dot(dd, mm)
        root = (Bq * Bq - Aq * (_dot(mm, mm) - rr * rr)).sqrt()
        sv = torch.where((-Bq - root) / Aq >= 1, (-Bq - root) / Aq, (-Bq + root) / Aq)
        q = sv.unsqueeze(-1) * dd + mm
        l = _mv(R[k].transpose(1, 2), q) / rr.unsqueeze(-1)
        ny, nx = ts.shape
        col = _bilinear(ts, (l[:, 0] + 1) * 0.5 * (nx - 1), (l[:, 1] + 1) * 0.5 * (ny - 1))
        g, = torch.autograd.grad((col * wt[e].reshape(-1)[px]).sum(), x)
        images.append(colour_g.index_copy(0, px, col.detach()).view(H, Wd).cpu())
        grads.append(g)
    g = torch.cat(grads)
    return dict(image=torch.stack(images), g_x=torch.cat([g, torch.zeros(len(g), 6, dtype=g.dtype, device=dev)], 1).T.cpu())


def _exact_fit(case, seed):
    rec, w0 = _records(case, seed)
    rec = torch.tensor(rec).double()
    w = torch.tensor(W.f32(w0)).float()
    p = w.bfloat16().double().requires_grad_()
    h, o = rec[:, :7], 0
    for a, b, last in ((7, 64, 0), (64, 64, 0), (64, 3, 1)):
        h = h @ p[o:o + a * b].view(b, a).T + p[o + a * b:o + a * b + b]
        h, o = (h if last else torch.relu(h)), o + a * b + b
    e = h - (rec[:, 7:10] - rec[:, 4:7])
    hb = float(np.float32(0.05))
    loss = torch.where(e.abs() > hb, 2 * hb * e.abs() - hb * hb, e * e).sum() / len(rec)
    g, = torch.autograd.grad(loss, p)
    # one Adam step from zero moments (the update's direction is that of each
    # gradient's sign, so the weights are compared with the start's alone)
    return dict(loss=loss.detach().view(1), grad=g, w=None, m=0.1 * g, v=0.001 * g * g)


def exact(case, seed):
    if case["kind"] == "fit":
        return _exact_fit(case, seed)
    if case["kind"] == "camera":
        return _exact_camera(case, seed)
    if case["kind"] == "solve":
        return None   # up to a thousand sweeps a step
    if case["kind"] == "train" and case["model"] == "chains":
        return None   # a hundred steps of sweeps over up to 33 visits, and their gradient: minutes
    return _exact_rollout(case, seed)
