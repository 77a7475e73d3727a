"""GPU tests of the one-wave kernels (block layout, exact mode) against the
workgroup kernels (block_threads asks for the latter): finish times and statistics bit
for bit, at the edges of the wave kernels' lists (256, exact mode 512 active and 512
pending flows, 64 finished flows at once), where a part is handed over in the middle
of an event, and when the run is advanced in pieces across the hand-over."""

import sys

import numpy as np
import pytest

from oracle import sim as osim
from workloads.program import Barrier, PathFlow, Program, Scenario, Topology
from workloads.rng import Stream

pytestmark = pytest.mark.gpu

SAME = ("events", "solves", "rounds", "flows_swept", "incidences_swept", "active_swept", "pending_swept",
        "reselected", "completed_flows", "links_swept", "launch_events")


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_01616_amd import netsim as ns
    from paper_2505_01616_amd import program as prog
    return ns, prog


def _say(*a):
    print(*a, file=sys.stderr, flush=True)


def _release(n, lagged, latency=False, links=40, seed=9, deg=6):
    """A flow, then n flows released by its end (all at once, or each at an
    instant of its own), then a barrier over them and 150 zero-byte flows
    that finish together, each with a flow after it."""
    u = Stream(seed, "wave-release").u01(8 * n + 1000)
    caps = 1.0 + np.floor(9.0 * u[:links])
    topo = Topology(kind="explicit", capacities=caps)
    if latency:
        topo.latencies = 0.25 * u[links:2 * links]
    sc = Scenario(topo)
    first = sc.add(PathFlow([0], 8.0))
    ids = []
    for i in range(n):
        r = u[100 + 8 * i:108 + 8 * i]
        path = sorted({int(x * links) for x in r[:1 + int(deg * r[6])]})
        ids.append(sc.add(PathFlow(path, float(1 + int(40 * r[7])), lag=float(1.0 + 7.0 * r[5]) if lagged else 0.0,
                                   after=(first,))))
    b = sc.add(Barrier(after=tuple(ids)))
    for i in range(150):
        z = sc.add(Barrier(after=(b,)))
        sc.add(PathFlow([i % links], 2.0 + i % 7, after=(z,)))
    return Program(f"release-{n}", [sc])


@pytest.mark.parametrize("latency", [False, True])
@pytest.mark.parametrize("n,lagged", [(255, False), (256, False), (257, False), (700, False), (511, True),
                                      (512, True), (513, True), (1500, True)])
def test_hand_over(n, lagged, latency):
    ns, pr = _gpu()
    program = _release(n, lagged, latency)
    _say(f"test_hand_over n={n} lagged={lagged} latency={latency}")
    a, sa = pr.run_program(program, ns.make_options())
    b, sb = pr.run_program(program, ns.make_options(block_threads=512))
    assert np.array_equal(a[0], b[0])
    for k in SAME:
        assert sa[k] == sb[k], (k, sa[k], sb[k])
    want = osim.run_scenario(program.scenarios[0]).finish
    assert np.max(np.abs(a[0] - want) / want) < 1e-9


@pytest.mark.parametrize("latency", [False, True])
@pytest.mark.parametrize("n,lagged", [(120, False), (129, False), (511, False), (512, False), (513, False),
                                      (700, False), (512, True), (513, True), (1500, True)])
def test_exact_hand_over(n, lagged, latency):
    """Exact mode: bit for bit the oracle, in one run and advanced in pieces
    across the hand-over, with the workgroup kernel's counters."""
    ns, pr = _gpu()
    program = _release(n, lagged, latency)
    _say(f"test_exact_hand_over n={n} lagged={lagged} latency={latency}")
    want = osim.run_scenario(program.scenarios[0])
    a, sa = pr.run_program(program, ns.make_options(exact=1))
    b, sb = pr.run_program(program, ns.make_options(exact=1, block_threads=512))
    assert np.array_equal(a[0], want.finish) and np.array_equal(b[0], want.finish)
    for k in SAME:
        assert sa[k] == sb[k], (k, sa[k], sb[k])
    assert (sa["events"], sa["solves"], sa["rounds"]) == (want.events, want.solves, want.iterations)
    ld = pr.load_program(program, ns.make_options(exact=1))
    try:
        for _ in range(200):
            ns.netsim_advance(ld.handle, max_events=41)
            if ns.netsim_get_stats(ld.handle)["complete"]:
                break
        assert np.array_equal(ns.netsim_get_finish(ld.handle), want.finish)
    finally:
        ld.close()


@pytest.mark.parametrize("deg", [1, 2, 3, 4, 5, 6, 7])
def test_path_lengths(deg):
    """The longest path chooses the loop (2, 4 or 6 links; longer: the workgroup kernel)."""
    ns, pr = _gpu()
    program = _release(120, False, True, links=60, deg=deg)
    paths = [f.path for f in program.scenarios[0].ops if isinstance(f, PathFlow)]
    _say(f"test_path_lengths deg={deg} longest={max(map(len, paths))}")
    assert max(map(len, paths)) == deg
    a, sa = pr.run_program(program, ns.make_options())
    b, sb = pr.run_program(program, ns.make_options(block_threads=512))
    assert np.array_equal(a[0], b[0])
    for k in SAME:
        assert sa[k] == sb[k], (k, sa[k], sb[k])
    want = osim.run_scenario(program.scenarios[0]).finish
    assert np.max(np.abs(a[0] - want) / want) < 1e-9


@pytest.mark.parametrize("history", [0, 8])
@pytest.mark.parametrize("n,lagged", [(40, False), (300, False), (600, True)])
def test_pieces_and_rollback(n, lagged, history):
    """Advancing by events (the launch's limit counts both kernels' events)
    equals one run, before and after a start moves into the past."""
    ns, pr = _gpu()
    program = _release(n, lagged)
    _say(f"test_pieces_and_rollback n={n} lagged={lagged} history={history}")
    want, _ = pr.run_program(program, ns.make_options(block_threads=512))
    later = _release(n, lagged)
    op = later.scenarios[0].ops[20]
    op.lag = op.lag + 3.5
    want2, _ = pr.run_program(later, ns.make_options(block_threads=512))
    ld = pr.load_program(program, ns.make_options(history_mb=history))
    try:
        events = 0
        for _ in range(2000):
            ns.netsim_advance(ld.handle, max_events=7)
            st = ns.netsim_get_stats(ld.handle)
            assert st["launch_events"] <= 7 and st["events"] == events + st["launch_events"]
            events = st["events"]
            if st["complete"]:
                break
        assert np.array_equal(ns.netsim_get_finish(ld.handle), want[0])
        ns.netsim_update_start(ld.handle, 20, op.lag)
        ns.netsim_advance(ld.handle)
        assert np.array_equal(ns.netsim_get_finish(ld.handle), want2[0])
    finally:
        ld.close()


def _followed(n, latency):
    """n flows and 90 zero-byte flows that end at one instant, each followed by
    a computation, a second one after it and a lagged flow after that, and by
    a lagged flow of its own: every release lies after its predecessor's end
    by a lag of its own."""
    topo = Topology(kind="explicit", capacities=np.full(n, 2.0))
    if latency:
        topo.latencies = 0.25 + 0.125 * (np.arange(n) % 5)
    sc = Scenario(topo)
    first = sc.add(PathFlow([0], 2.0))
    ends = [sc.add(PathFlow([i], 20.0, after=(first,))) for i in range(n)]
    at = sc.add(Barrier(lag=64.0, after=(first,)))
    ends += [sc.add(Barrier(after=(at,))) for _ in range(90)]
    for i, f in enumerate(ends):
        c = sc.add(Barrier(lag=0.001 * (1 + i), after=(f,)))
        d = sc.add(Barrier(lag=0.5, after=(c,)))
        sc.add(PathFlow([i % n], 3.0, lag=0.25, after=(d,)))
        sc.add(PathFlow([i % n], 2.0 + i % 7, lag=1.0 + 0.125 * (i % 5), after=(f,)))
    return Program(f"followed-{n}", [sc])


@pytest.mark.parametrize("latency", [False, True])
@pytest.mark.parametrize("n", [64, 65, 128, 200])
def test_many_ends_followed_by_lags(n, latency):
    """More flows end in one event than the newest 64 that the log keeps in
    shared memory, and everything after them counts from their ends: exact
    mode bit for bit the oracle, whole and in pieces; the default solver bit
    for bit the workgroup kernel's."""
    ns, pr = _gpu()
    program = _followed(n, latency)
    _say(f"test_many_ends_followed_by_lags n={n} latency={latency}")
    want = osim.run_scenario(program.scenarios[0])
    a, sa = pr.run_program(program, ns.make_options(exact=1))
    assert np.array_equal(a[0], want.finish)
    assert (sa["events"], sa["solves"], sa["rounds"]) == (want.events, want.solves, want.iterations)
    ld = pr.load_program(program, ns.make_options(exact=1))
    try:
        for _ in range(400):
            ns.netsim_advance(ld.handle, max_events=13)
            if ns.netsim_get_stats(ld.handle)["complete"]:
                break
        assert np.array_equal(ns.netsim_get_finish(ld.handle), want.finish)
    finally:
        ld.close()
    b, sb = pr.run_program(program, ns.make_options())
    c, sc = pr.run_program(program, ns.make_options(block_threads=512))
    assert np.array_equal(b[0], c[0])
    for k in SAME:
        assert sb[k] == sc[k], (k, sb[k], sc[k])
    assert np.max(np.abs(b[0] - want.finish) / want.finish) < 1e-9


def test_phase_times_of_a_part_handed_over():
    """The phase timers count both kernels' time: 400 flows one after another
    in the one-wave kernel, then 300 at once, which it hands over."""
    ns, pr = _gpu()
    _say("test_phase_times_of_a_part_handed_over")
    sc = Scenario(Topology(kind="explicit", capacities=np.full(8, 4.0)))
    last = sc.add(PathFlow([0], 1.0))
    for i in range(400):
        last = sc.add(PathFlow([i % 8], 1.0 + i % 3, after=(last,)))
    for i in range(300):
        sc.add(PathFlow([i % 8], 2.0, after=(last,)))
    program = Program("phases", [sc])
    _, s = pr.run_program(program, ns.make_options(debug=2))
    _, t = pr.run_program(program, ns.make_options())
    assert s["events"] == t["events"] >= 402
    # most of the run is in a phase (the rest: reading and writing positions)
    assert sum(s["phase_seconds"]) > 0.5 * s["device_seconds"], (s["phase_seconds"], s["device_seconds"])


@pytest.mark.parametrize("n", [448, 449, 512])
def test_exact_hand_over_with_many_links(n):
    """Scenarios of more than 1,024 links leave the one-wave kernel at 448
    active flows: bit for bit the oracle on both sides of the line."""
    ns, pr = _gpu()
    program = _release(n, False, links=4000)
    used = {l for f in program.scenarios[0].ops if isinstance(f, PathFlow) for l in f.path}
    _say(f"test_exact_hand_over_with_many_links n={n} links={len(used)}")
    assert len(used) > 1024
    want = osim.run_scenario(program.scenarios[0])
    a, sa = pr.run_program(program, ns.make_options(exact=1))
    assert np.array_equal(a[0], want.finish)
    assert (sa["events"], sa["solves"], sa["rounds"]) == (want.events, want.solves, want.iterations)
