"""The saved working sets' offsets, on the host, at the sizes that are run: 2048
uneven chains of 2 to 32 bodies over 120 steps (every working set kept), 333 of
them by segments, and 16384 over 500 steps, whose buffer of 6.4e10 floats is
past 32-bit offsets.  Every step of every env, its sweeps' history and its tail
lie in the env's own block, first and last env included, and the forward and
reverse kernels agree on the layout."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_1611_01652_amd import workloads as W
from test_kernel_host_fp64 import ROOT, _desc64, _store

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "kernel_host", "working_sets.cpp")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("ws") / "libworking_sets.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-o", out, SRC], cwd=ROOT)
    lib = C.CDLL(out)
    lib.kw_check.restype = C.c_longlong
    return lib


def _chains(n, T):
    rng = np.random.default_rng([n, 2, 32])
    return W.uneven_chains(n_envs=n, T=T, sizes=W.chain_sizes(n, rng, lo=2, hi=32))


def _segments(w):
    w.ckpt_every = 25
    return _store(w, "segment")


def _episodes(n):
    w = W.quadruped(n_envs=n, T_min=1, T_max=61, mlp_w=W.mlp_init(zero_output=False, out_scale=0.1))
    w.ckpt_every = 7
    return _store(w, "trajectory")


@pytest.mark.parametrize("maker,floor", [
    (lambda: _store(_chains(2048, 120), "trajectory"), 1e9),
    (lambda: _segments(_chains(333, 75)), 1e7),
    (lambda: _store(_chains(16384, 500), "trajectory"), 4e9),
    (lambda: _episodes(70), 1e5),                            # episode lengths of their own
    (lambda: _segments(W.servo_chains(12, 60)), 1e5),
])
def test_every_working_set_lies_in_its_env_s_block(lib, maker, floor):
    d, keep = _desc64(maker())
    total, bad = C.c_longlong(), C.c_longlong()
    assert lib.kw_check(C.byref(d), C.byref(total), C.byref(bad)) == 0, bad.value
    assert total.value > floor
