"""TEST INFRASTRUCTURE ONLY: jointed robots with more contacts than the
narrowest team has lanes, and the count of their contacts.

A wave holds its constraints' rows in registers only while every env has at
most one joint per pair of lanes and one placed contact per lane; these models
are past that at a narrow width and within it at a wide one."""
from __future__ import annotations

import numpy as np

from paper_1611_01652_amd import workloads as W


def lying_chains(sizes, T, per_body=2, depth=0.05, seed_salt=1, servo=False, tol=0.0, net=None):
    """Uneven chains of the given body counts, lowered until their lowest
    sphere reaches `depth` below the ground and straightened towards it, with
    `per_body` ground spheres on each body.  servo: hinges are servos; tol:
    each step is solved to that residual, with the learned start if net."""
    w = W.uneven_chains(n_envs=len(sizes), T=T, seed_salt=seed_salt, sizes=np.asarray(sizes))
    if servo:
        w = W.with_servos(w, gain=20.0, torque=5.0, vmax=3.0,
                          targets=W.servo_targets(T, w.n_joints, seed_salt=seed_salt, amp=0.3, hold=5))
    body = np.repeat(np.arange(w.n_bodies), per_body)
    r = np.asarray(w.sphere_radius, np.float64)
    off = np.zeros((w.n_bodies, per_body, 3))
    flags = np.zeros((w.n_bodies, per_body), np.int32)
    rad = np.repeat(r[:, None], per_body, 1)
    flags[:, 0] = W.SPHERE_GROUND | W.SPHERE_PAIR
    for k in range(1, per_body):   # smaller ones beside the first, as low
        off[:, k, k % 2] = 0.3 * r * (-1) ** k
        rad[:, k] = 0.95 * r
        flags[:, k] = W.SPHERE_GROUND
    w.sphere_body = body.astype(np.int32)
    w.sphere_offset = W.f32(off.reshape(-1, 3))
    w.sphere_radius = W.f32(rad.reshape(-1))
    w.sphere_flags = flags.reshape(-1)
    w.env_sphere_off = (np.asarray(w.env_body_off) * per_body).astype(np.int32)
    # (the chains' pitch angles lift them off the ground: a body rests `depth`
    # to 1.5 `depth` deep instead, its joints pulling it to its neighbours)
    rng = np.random.default_rng(seed_salt)
    w.x0 = w.x0.copy()
    w.x0[:, 2] = r - depth * rng.uniform(1.0, 1.5, w.n_bodies)
    w.x0 = W.f32(w.x0)
    if tol:
        w.warm = 1.0
        w.extra = dict(w.extra or {}, solve=dict(mode=1, tol=float(tol), max_iters=400))
        if net is not None:
            w.extra["ws"] = dict(w=np.asarray(net, np.float64), fb_iters=5, fb_tol=1e-3)
    return w


def first_step_contacts(w):
    """[E] contacts that are active in the first step: candidates with a gap
    below the margin at the initial state (jointed bodies do not touch)."""
    x = np.asarray(w.x0, np.float64)
    R = x[:, 3:12].reshape(-1, 3, 3)
    body = np.asarray(w.sphere_body)
    c = x[body, :3] + np.einsum("sij,sj->si", R[body], np.asarray(w.sphere_offset, np.float64))
    r = np.asarray(w.sphere_radius, np.float64)
    n = np.zeros(w.n_envs, int)
    for e in range(w.n_envs):
        s = np.arange(w.env_sphere_off[e], w.env_sphere_off[e + 1])
        if w.ground:
            g = s[(w.sphere_flags[s] & W.SPHERE_GROUND) != 0]
            n[e] += int((c[g, 2] - r[g] < w.spec_margin).sum())
        p = s[(w.sphere_flags[s] & W.SPHERE_PAIR) != 0]
        j = range(w.env_joint_off[e], w.env_joint_off[e + 1])
        joined = {frozenset((int(w.joint_parent[k]), int(w.joint_child[k]))) for k in j}
        for i in range(len(p)):
            for k in range(i + 1, len(p)):
                a, b = p[i], p[k]
                if frozenset((int(body[a]), int(body[b]))) in joined:
                    continue
                n[e] += int(np.linalg.norm(c[a] - c[b]) - r[a] - r[b] < w.spec_margin)
    return n


def capacity(w):
    """[E] contacts an env has row slots for: every candidate when few, else
    two per body and four."""
    nb = np.diff(w.env_body_off)
    out = np.zeros(w.n_envs, int)
    for e in range(w.n_envs):
        s = np.arange(w.env_sphere_off[e], w.env_sphere_off[e + 1])
        G = int((w.sphere_flags[s] & W.SPHERE_GROUND != 0).sum()) if w.ground else 0
        k = int((w.sphere_flags[s] & W.SPHERE_PAIR != 0).sum())
        nj = int(w.env_joint_off[e + 1] - w.env_joint_off[e])
        out[e] = min(G + k * (k - 1) // 2 - nj, 2 * nb[e] + 4)
    return out
