"""GPU tests of the single rate solve through a handle (netsim_solve_once,
default solver) against the oracle: link state in shared memory up to its
limit and in global memory beyond it, subsets of the flows active (links that
only inactive flows cross), one flow, and paths too long for a path record.

Tolerance: a rate is a quotient of a residual (a capacity less at most 1,000
rates, each rounded to 2^-61 of the largest capacity) and a count; shares
within 1e-12 of a level freeze with it.  So 1e-11 relative covers both sides."""

import sys

import numpy as np
import pytest

from oracle import sim as osim
from workloads.program import PathFlow, Program, Scenario, Topology
from workloads.rng import Stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("links,flows,deg,share", [
    (5554, 9000, 6, 1.0), (5555, 9000, 6, 0.3), (5560, 9000, 6, 0.3), (1, 40, 1, 1.0), (64, 700, 3, 0.5),
    (3, 1, 2, 1.0), (300, 4100, 6, 1.0), (40, 300, 9, 0.7)])
def test_solve_once(links, flows, deg, share):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_01616_amd import netsim as ns
    from paper_2505_01616_amd import program as prog
    print(f"test_solve_once links={links} flows={flows} deg={deg} share={share}", file=sys.stderr, flush=True)
    u = Stream(links * 10007 + flows, "solve-once").u01(links + flows * (deg + 2))
    caps = 1.0 + 9.0 * u[:links]
    sc = Scenario(Topology(kind="explicit", capacities=caps))
    paths = []
    for i in range(flows):
        r = u[links + i * (deg + 2):links + (i + 1) * (deg + 2)]
        # every link is crossed by some flow, so all of them count towards the limit
        paths.append(sorted({i % links} | {int(x * links) for x in r[:int(deg * r[deg])]}))
        sc.add(PathFlow(paths[-1], 1.0))
    active = np.nonzero(u[links + deg + 1::deg + 2][:flows] <= share)[0]
    poff = np.concatenate([[0], np.cumsum([len(p) for p in paths])]).astype(np.int64)
    want = osim.solve_rates(caps, poff, np.concatenate(paths).astype(np.int32), active)
    # one part, so that all links belong to one solve
    ld = prog.load_program(Program("solve", [sc]), ns.make_options(single_clock=1))
    try:
        got = ns.netsim_solve_once(ld.handle, 0, active)
        again = ns.netsim_solve_once(ld.handle, 0, active[: max(1, len(active) // 3)])
    finally:
        ld.close()
    assert len(got) == len(want) and np.max(np.abs(got - want) / want) < 1e-11
    want = osim.solve_rates(caps, poff, np.concatenate(paths).astype(np.int32), active[: max(1, len(active) // 3)])
    assert np.max(np.abs(again - want) / want) < 1e-11
