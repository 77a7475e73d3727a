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


def _case(links, flows, deg, equal, seed):
    """Random paths over `links` links; equal: every capacity the same and one
    flow per link (all links are bottlenecks of one level)."""
    u = Stream(seed, "solve-exact").u01(links + flows * (deg + 1))
    caps = np.full(links, 8.0) if equal else 1.0 + np.floor(1e3 * u[:links])
    paths = []
    for i in range(flows):
        r = u[links + i * (deg + 1):links + (i + 1) * (deg + 1)]
        paths.append([i % links] if equal else sorted({int(x * links) for x in r[:1 + int(deg * r[deg])]}))
    poff = np.concatenate([[0], np.cumsum([len(p) for p in paths])]).astype(np.int64)
    return caps, paths, poff, np.concatenate(paths).astype(np.int32)


# link state in shared and in global memory, more links than the lists hold
# (sweeps), paths beyond a record, more bottlenecks and touched links in a
# level than are listed, the smallest sizes that go by links
EXACT = [(300, 1023, 4, False), (300, 1024, 4, False), (40, 2000, 9, False), (4500, 6000, 6, False),
         (9000, 20000, 6, False), (9000, 20000, 7, False), (40000, 3000, 5, False), (7000, 7000, 1, True),
         (2, 1500, 2, False)]


@pytest.mark.parametrize("links,flows,deg,equal", EXACT)
def test_exact_by_links(links, flows, deg, equal):
    """Exact mode through a handle and on device arrays: bit for bit the
    oracle's rates, and the levels of the whole-GPU solve."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_01616_amd import netsim as ns
    from paper_2505_01616_amd import program as prog
    print(f"test_exact_by_links links={links} flows={flows} deg={deg} equal={equal}", file=sys.stderr, flush=True)
    caps, paths, poff, plink = _case(links, flows, deg, equal, links + flows + deg)
    want = osim.solve_rates(caps, poff, plink, np.arange(flows))
    sc = Scenario(Topology(kind="explicit", capacities=caps))
    for p in paths:
        sc.add(PathFlow(p, 1.0))
    stats = []
    for debug in (0, 32):  # by links where they fit; every level on the whole GPU
        ld = prog.load_program(Program("solve", [sc]), ns.make_options(exact=1, debug=debug))
        try:
            got = ns.netsim_solve_once(ld.handle, 0, np.arange(flows))
            stats.append([ns.netsim_get_stats(ld.handle)[k] for k in ("rounds", "flows_swept", "incidences_swept",
                                                                       "links_swept")])
            part = np.arange(0, flows, 3)  # a subset: other flows are listed on the links too
            some = ns.netsim_solve_once(ld.handle, 0, part)
        finally:
            ld.close()
        assert np.array_equal(got, want)
        assert np.array_equal(some, osim.solve_rates(caps, poff, plink, part))
    assert stats[0] == stats[1]
    d = [torch.from_numpy(x).cuda() for x in (caps, poff.astype(np.int32), plink)]
    rates = torch.full((flows,), -1.0, dtype=torch.float64, device="cuda")
    status = torch.full((2,), 7, dtype=torch.int64, device="cuda")
    for _ in range(2):
        ns.netsim_solve_rates_noalloc(0, links, d[0].data_ptr(), flows, d[1].data_ptr(), d[2].data_ptr(),
                                      rates.data_ptr(), status.data_ptr(), torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert status.tolist() == [ns.OK, stats[0][0]]
        assert np.array_equal(rates.cpu().numpy(), want)


@pytest.mark.parametrize("levels,limit,ok", [(1, 1, True), (2, 1, False), (8, 2, True), (65, 2, True), (66, 2, False),
                                             (66, 66, True), (129, 66, True), (130, 66, False)])
def test_exact_watchdog_of_wide_solves(levels, limit, ok):
    """max_rounds in an exact solve of 16,384 flows and more is looked at after
    levels 2, 66, 130, ...: a solve that ends before the next look passes,
    by links as on the whole GPU (debug bit 5)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_01616_amd import netsim as ns
    from paper_2505_01616_amd import program as prog
    print(f"test_exact_watchdog levels={levels} limit={limit}", file=sys.stderr, flush=True)
    flows = 16384
    caps = 100.0 + np.arange(levels)  # a flow crosses one link: a level per link
    sc = Scenario(Topology(kind="explicit", capacities=caps))
    for i in range(flows):
        sc.add(PathFlow([i % levels], 1.0))
    count = np.bincount(np.arange(flows) % levels)
    assert len(np.unique(caps / count)) == levels
    for debug in (0, 32):
        ld = prog.load_program(Program("watchdog", [sc]), ns.make_options(exact=1, max_rounds=limit, debug=debug))
        try:
            if ok:
                got = ns.netsim_solve_once(ld.handle, 0, np.arange(flows))
                assert np.array_equal(got, (caps / count)[np.arange(flows) % levels])
                assert ns.netsim_get_stats(ld.handle)["rounds"] == levels
            else:
                with pytest.raises(ns.NetsimError, match="watchdog"):
                    ns.netsim_solve_once(ld.handle, 0, np.arange(flows))
        finally:
            ld.close()
