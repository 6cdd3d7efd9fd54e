"""TEST INFRASTRUCTURE ONLY: lanes_run.py's runs on jointed robots whose
constraints do not fit the lanes (the sweeps then walk the visit list), see
tests/test_kernel_host_listed.py."""
import sys

import lanes_run as R
from contact_models import lying_chains
from paper_1611_01652_amd import workloads as W

R.CASES.update({
    "listed": lambda: lying_chains([5, 5], 8),
    "listed-replay": lambda: R._store(lying_chains([5, 4], 6), "replay"),
    "listed-segment": lambda: R._store(lying_chains([5, 5], 6), "segment"),
    "listed-servo": lambda: lying_chains([5, 4], 6, servo=True),
    # one env of the wave fits its lanes, the other does not
    "listed-mixed": lambda: lying_chains([2, 5], 6),
    # more joints than pairs of lanes in the widest team
    "listed-40": lambda: lying_chains([40], 2, per_body=1),
})
R.SOLVE_CASES.update({
    "listed-solve": lambda: lying_chains([5, 4], 3, tol=1e-5),
    "listed-learned": lambda: lying_chains([5, 5], 3, tol=1e-5, net=W.wsn_init(seed_salt=2, scale=0.2)),
})

if __name__ == "__main__":
    sys.exit(R.main())
