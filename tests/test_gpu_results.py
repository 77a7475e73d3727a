"""GPU tests of the results gathered on the device: finish times in id order, the
largest of each scenario and the counts, where scenarios end at, beside and far from
the 2048 flows a workgroup gathers, after a whole run, a part of one and a run again."""

import sys

import numpy as np
import pytest

from oracle import sim as osim
from workloads.program import PathFlow, Program, Scenario, Topology

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1,), (2048,), (2049,), (2047, 1, 1, 2047), (3, 2500, 1, 60, 1400, 400, 2048, 5)])
def test_results(sizes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_01616_amd import netsim as ns
    from paper_2505_01616_amd import program as prog
    print("test_results", sizes, file=sys.stderr, flush=True)
    scenarios = []
    for k, n in enumerate(sizes):
        sc = Scenario(Topology(kind="explicit", capacities=np.array([1.0, 2.0, 3.0, 5.0])))
        for i in range(n):  # up to 7 instants at which flows end, per scenario times of its own
            sc.add(PathFlow([(i + k) % 4], float(1 + i % 7 + k)))
        scenarios.append(sc)
    program = Program("results", scenarios)
    want = np.concatenate([osim.run_scenario(sc).finish for sc in scenarios])
    off = np.concatenate([[0], np.cumsum(sizes)])

    def check(ld):
        fin = ns.netsim_get_finish(ld.handle)
        st = ns.netsim_get_stats(ld.handle)
        done = ~np.isnan(fin)
        # eight-byte values moved, none computed: equal bit for bit
        most = [np.max(fin[a:b], initial=0.0, where=done[a:b]) for a, b in zip(off[:-1], off[1:])]
        assert np.array_equal(ns.netsim_get_makespan(ld.handle, len(sizes)), most)
        assert st["completed_flows"] == done.sum() and st["complete"] == done.all()
        assert st["sim_time"] == max(most)  # the last event ends a flow
        assert np.max(np.abs(fin[done] - want[done]) / want[done], initial=0.0) < 1e-9
        return fin

    ld = prog.load_program(program, ns.make_options())
    try:
        ns.netsim_advance(ld.handle, max_events=2)  # the starts, then one instant of ends in each part
        part = check(ld)
        assert np.isnan(part).any() == (len(part) > 1) and not np.isnan(part).all()
        ns.netsim_run(ld.handle)
        a = check(ld)
        ns.netsim_advance(ld.handle)
        assert np.array_equal(a, check(ld))
        ns.netsim_run(ld.handle)
        assert np.array_equal(a, check(ld)) and not np.isnan(a).any()
    finally:
        ld.close()
