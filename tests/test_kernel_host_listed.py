"""Sweeps over the visit list with hinges, on the host (as
test_kernel_host_lanes.py: whole waves of lanes in FP64 under three lane
schedules, accesses checked by AddressSanitizer, equal to the FP64 oracle).

A jointed env with more contacts than its team has lanes, or more joints than
pairs of lanes, walks the visit list: forward, the reverse from replays and
from saved working sets, servo motors, and sweeps to a tolerance with a plain
and a learned start (of contacts that are really placed).  The same models at
a width that holds every row in registers give the same results."""
import json
import os
import subprocess
import sys

import pytest

from contact_models import capacity, first_step_contacts, lying_chains
from test_kernel_host_lanes import KH, lanes_lib   # noqa: F401


def _run(lib_rt, team, teams_per_wave, cases):
    lib, rt = lib_rt
    env = dict(os.environ, LD_PRELOAD=rt, ASAN_OPTIONS="detect_leaks=0")
    p = subprocess.run([sys.executable, os.path.join(KH, "lanes_listed_run.py"), lib, str(-team),
                        str(teams_per_wave)] + cases, capture_output=True, text=True, env=env, timeout=900)
    assert "AddressSanitizer" not in p.stderr, p.stderr[-3000:]
    assert p.returncode == 0, p.stderr[-3000:]
    rows = [json.loads(line) for line in p.stdout.splitlines() if line.startswith("{")]
    assert [r["case"] for r in rows] == cases, p.stdout
    return rows


FIXED = ["listed", "listed-replay", "listed-segment", "listed-servo", "listed-mixed"]
SOLVE = ["listed-solve", "listed-learned"]


# 5 bodies: 4 joints, 10 contacts (4: 3 and 8); on 2 and 4 lanes the joints are
# too many, on 8 the contacts, on 16 and more every row is held
@pytest.mark.parametrize("team,teams_per_wave,cases", [
    (2, 2, ["listed", "listed-servo"]),
    (4, 2, ["listed-replay", "listed-segment", "listed-learned"]),
    (8, 2, FIXED),
    (8, 2, SOLVE),
    (16, 2, FIXED + SOLVE),
    (64, 1, ["listed-40"]),
])
def test_listed_and_held_waves_equal_the_oracle(lanes_lib, team, teams_per_wave, cases):   # noqa: F811
    for sizes, lanes in (([5, 5], 8), ([40], 32)):
        w = lying_chains(sizes, 1, per_body=2 if sizes[0] == 5 else 1)
        n = first_step_contacts(w)
        assert (n > lanes).all() and (n <= capacity(w)).all()
    for r in _run(lanes_lib, team, teams_per_wave, cases):
        assert "error" not in r, r
        assert r["schedules_agree"], r
        assert r["counts_agree"], r
        assert r["max_rel_diff"] < 1e-8, r
