"""The work a user of the simulator has it do, as cases to time and compare.

Each case is one pass through the public entry points (the Python binding of
include/netsim.h): complete simulations of collectives, of a 3D-parallel
step, of a training-step trace issued on streams, of expert-parallel
all-to-alls, of a batch of what-if scenarios and of a degraded fat-tree in
exact mode; a run advanced in steps with a start moved into its past; and
single max-min rate solves, through a handle and on device arrays.  Sizes
are those of the workloads of workloads/, README.md and bench.py, or lie
around them.  Outputs are every flow's finish time (and every scenario's
makespan) or every flow's rate.

``exact`` computes the same results in plain numpy: its own routing,
decomposition, event loop and progressive filling in 64 bits.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_01616_amd import netsim as ns

MiB, GiB = float(1 << 20), float(1 << 30)
INF = math.inf


def listed():
    return [
        # one ring all-reduce of 64 GPUs, 126 chained steps: the smallest
        # simulation, one operation looked up before a job is placed
        dict(name="ring64", kind="ring", ranks=64, mode="chained", mib=256.0, exact=0),
        # one 3D-parallel step on 128 GPUs: tensor-parallel rings inside the
        # servers, pipeline sends, gradient rings; many independent parts
        dict(name="step128", kind="step", tp_reps=24, pp=4, dp=4, micro=8, exact=0),
        # a training step as the tracer delivers it: 128 GPUs, computations,
        # collectives and sends on streams; one part, tens of active flows
        dict(name="trace128", kind="trace", tp=8, pp=4, dp=4, micro=8, layers=4, allreduce="ring",
             latency_us=0.0, exact=0),
        # the same front end with tree all-reduce and link latencies, advanced
        # in steps; then a computation turns out longer and the simulation
        # goes back to before it (the throughput history kept)
        dict(name="rollback64", kind="rollback", tp=8, pp=4, dp=2, micro=6, layers=2, allreduce="tree",
             latency_us=2.0, step_events=1000, history_mb=64),
        # eight expert-parallel groups of 32 ranks (256 GPUs) that share their
        # servers' fabric: dispatch, then combine
        dict(name="a2a_256gpu", kind="a2a", groups=8, ranks=32, phases=2, exact=0),
        # eight groups of 56 ranks: a wide all-to-all phase, every flow of it
        # released at once and most finishing at instants of their own
        dict(name="a2a_448gpu", kind="a2a", groups=8, ranks=56, phases=1, exact=0),
        # what-if batch: 64 scenarios of a 4096-GPU rail fabric (parallelism,
        # NIC rate and oversubscription vary), aggregated collectives
        dict(name="whatif64", kind="whatif", scenarios=64, servers=512),
        # gradient rings over a fat-tree with a tenth of its cables degraded
        # and background transfers, in the arithmetic of the sequential program
        dict(name="fattree_exact", kind="fattree", groups=4, ranks=32, background=200, exact=1),
        # the rates of one instant: every flow of an all-to-all phase on 4096
        # GPUs at once (64 groups of 64 ranks)
        dict(name="solve_wide", kind="solve", groups=64, ranks=64, exact=0),
        # the same instant in exact mode
        dict(name="solve_wide_exact", kind="solve", groups=64, ranks=64, exact=1),
        # rates on arrays that the caller holds on the GPU (a serving loop):
        # one group's all-to-all of 16 ranks, and eight groups of 64
        dict(name="noalloc_small", kind="noalloc", groups=1, ranks=16),
        dict(name="noalloc_wide", kind="noalloc", groups=8, ranks=64),
    ]


def draw(rng):
    """One more case of the same ranges; none costs more than a2a_448gpu."""
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["ring", "step", "trace", "rollback", "a2a", "whatif", "fattree", "solve", "noalloc"])
    if kind == "ring":
        # a long chained ring amplifies rounding (one edge carries several
        # steps at once): beyond 64 ranks in exact mode only
        p, mode = log(5, 160), rng.choice(["chained", "flat", "aggregated"])
        return dict(kind=kind, ranks=p, mode=mode,
                    mib=float(round(math.exp(rng.uniform(math.log(1.0), math.log(4096.0))), 2)),
                    exact=1 if p > 64 and mode == "chained" else rng.choice([0, 0, 1]))
    if kind == "step":
        return dict(kind=kind, tp_reps=rng.randint(1, 24), pp=rng.choice([2, 3, 4, 5]), dp=rng.randint(2, 6),
                    micro=rng.randint(1, 9), exact=rng.choice([0, 0, 1]))
    if kind == "trace":
        return dict(kind=kind, tp=rng.choice([2, 4, 8]), pp=rng.randint(1, 4), dp=rng.randint(1, 5),
                    micro=rng.randint(1, 8), layers=rng.randint(1, 4), allreduce=rng.choice(["ring", "tree"]),
                    latency_us=rng.choice([0.0, round(rng.uniform(0.5, 5.0), 2)]), exact=rng.choice([0, 0, 1]))
    if kind == "rollback":
        return dict(kind=kind, tp=rng.choice([2, 4, 8]), pp=rng.randint(2, 4), dp=rng.randint(1, 3),
                    micro=rng.randint(2, 6), layers=rng.randint(1, 3), allreduce=rng.choice(["ring", "tree"]),
                    latency_us=rng.choice([0.0, round(rng.uniform(0.5, 5.0), 2)]),
                    step_events=log(200, 4000), history_mb=rng.choice([0, 16, 64]))
    if kind == "a2a":
        return dict(kind=kind, groups=rng.randint(2, 8), ranks=log(6, 38), phases=rng.randint(1, 2), exact=0)
    if kind == "whatif":
        return dict(kind=kind, scenarios=log(3, 96), servers=32 * rng.randint(1, 14))
    if kind == "fattree":
        return dict(kind=kind, groups=rng.randint(1, 8), ranks=log(6, 48), background=log(20, 300), exact=1)
    if kind == "solve":
        return dict(kind=kind, groups=log(1, 60), ranks=log(9, 64), exact=rng.choice([0, 1]))
    return dict(kind=kind, groups=rng.randint(1, 8), ranks=log(5, 63))


# ------------------------------------------------------------------ workloads
# A plan is one topology and list of operations per scenario.  Operations:
#   ("ring", mode, ranks, nbytes, lag, after)      all-reduce
#   ("a2a", ranks, matrix, lag, after)
#   ("sends", src, dst, nbytes, lag, deps)         deps[i]: indices of this batch
#   ("barrier", after)
# (`after`: operation indices) and, issued on streams,
#   ("compute", stream, seconds, waits)            waits: (operation, position)
#   ("allreduce", kind, ranks, streams, nbytes)
#   ("send", src, src_stream, dst, dst_stream, nbytes)

def _topology(kind, servers, per_leaf, nic, fabric, seed, **kw):
    t = dict(kind=kind, servers=servers, gpus=8, per_leaf=per_leaf, spines=0, pods=0, edges=0, aggs=0, ups=0,
             nv=900e9, nic=nic, fabric=fabric, seed=seed, degraded=np.zeros(0, np.int64), degraded_Bps=0.0,
             latency=0.0)
    t.update(kw)
    return t


def _ring_plan(case, rs):
    p = case["ranks"]
    servers = -(-p // 8)
    topo = _topology("leaf_spine", servers, 1, 50e9, 100e9, int(rs.randint(1 << 31)), spines=4)
    nbytes = case["mib"] * MiB * (1.0 + 0.1 * rs.rand())
    return [(topo, [("ring", case["mode"], np.arange(p), nbytes, 1e-4 * rs.rand(), [])])]


def _step_plan(case, rs):
    tp, dp, pp, micro = 8, case["dp"], case["pp"], case["micro"]
    servers = dp * pp
    topo = _topology("rail", servers, servers, 50e9, 100e9, int(rs.randint(1 << 31)), spines=8)
    ops = []
    for s in range(servers):
        after = []
        for rep in range(case["tp_reps"]):
            ops.append(("ring", "chained", np.arange(8 * s, 8 * s + 8), 32 * MiB, 50e-6 * rs.rand(), after))
            ops.append(("barrier", [len(ops) - 1]))
            after = [len(ops) - 1]
    src, dst, lag, deps = [], [], [], []
    for t in range(tp):
        for d in range(dp):
            rank = [t + tp * (d + dp * q) for q in range(pp)]
            at = {}
            for back in (0, 1):
                for m in range(micro):
                    for b in (range(pp - 1) if not back else range(pp - 2, -1, -1)):
                        a = []
                        prev = b - 1 if not back else b + 1
                        if 0 <= prev < pp - 1:
                            a.append(at[(back, prev, m)])
                        if m > 0:
                            a.append(at[(back, b, m - 1)])
                        if back and b == pp - 2 and m == 0:
                            a.append(at[(0, pp - 2, micro - 1)])
                        at[(back, b, m)] = len(src)
                        src.append(rank[b + back])
                        dst.append(rank[b + 1 - back])
                        lag.append(0.0 if a else 50e-6 * rs.rand())
                        deps.append(a)
    ops.append(("sends", np.array(src), np.array(dst), np.full(len(src), 16 * MiB), np.array(lag), deps))
    for t in range(tp):
        for q in range(pp):
            ranks = np.array([t + tp * (d + dp * q) for d in range(dp)])
            ops.append(("ring", "chained", ranks, 1 * GiB, 50e-6 * rs.rand(), []))
    return [(topo, ops)]


def _trace_plan(case, rs):
    """GPipe: forward and backward per micro-batch, stage and replica, an
    all-reduce after every layer, activations between the stages, gradient
    all-reduce and optimizer at the end.  Returns the plan and the operation
    whose duration the rollback case changes."""
    tp, pp, dp = case["tp"], case["pp"], case["dp"]
    n = tp * pp * dp
    servers = max(1, -(-n // 8))
    topo = _topology("rail", servers, servers, 50e9, 50e9, int(rs.randint(1 << 31)), spines=8,
                     latency=case["latency_us"] * 1e-6)
    ops, last = [], {}

    def add(op):
        ops.append(op)
        return len(ops) - 1

    def rank(t, d, s):
        return t + tp * (d + dp * s)

    def stage(d, s, seconds, recv):
        ranks = np.array([rank(t, d, s) for t in range(tp)])
        for t, r in enumerate(ranks):
            if recv is not None:
                last[r] = (add(("compute", 2 * r, 0.0, [recv[t]])), 0)
        for _ in range(case["layers"]):
            for r in ranks:
                last[r] = (add(("compute", 2 * r, seconds / case["layers"] * (0.9 + 0.2 * rs.rand()), [])), 0)
            if tp > 1:
                k = add(("allreduce", case["allreduce"], ranks, 2 * ranks, 16 * MiB))
                for t, r in enumerate(ranks):
                    last[r] = (k, t)
        return ranks

    def send_on(ranks, d, s):
        recv = []
        for t, a in enumerate(ranks):
            b = rank(t, d, s)
            add(("compute", 2 * a + 1, 0.0, [last[a]]))
            recv.append((add(("send", int(a), int(2 * a + 1), b, 2 * b + 1, 32 * MiB)), 1))
        return recv

    moved = None
    for back in (0, 1):
        recv = {}
        for m in range(case["micro"]):
            for d in range(dp):
                for s in (range(pp) if not back else reversed(range(pp))):
                    if back and m == case["micro"] // 2 and moved is None:
                        moved = len(ops) + (tp if recv.get((d, s, m)) is not None else 0)
                    ranks = stage(d, s, 2.4e-3 if back else 1.2e-3, recv.get((d, s, m)))
                    to = s - 1 if back else s + 1
                    if 0 <= to < pp:
                        recv[(d, to, m)] = send_on(ranks, d, to)
    for s in range(pp):
        for t in range(tp):
            ranks = np.array([rank(t, d, s) for d in range(dp)])
            waits = [[] for _ in ranks]
            if dp > 1:
                for r in ranks:
                    add(("compute", 2 * r + 1, 0.0, [last[r]]))
                k = add(("allreduce", case["allreduce"], ranks, 2 * ranks + 1, 512 * MiB))
                waits = [[(k, i)] for i in range(dp)]
            for i, r in enumerate(ranks):
                add(("compute", 2 * r, 0.5e-3 * (0.9 + 0.2 * rs.rand()), waits[i]))
    return [(topo, ops)], moved


def _zipf(rs, p):
    """Dispatch bytes of p ranks: every sender routes to the ranks with
    Zipf(1.2) popularity, mean 4 MiB."""
    w = (rs.permutation(p) + 1.0) ** -1.2
    m = np.tile(np.rint(4 * MiB * p * w / w.sum()), (p, 1))
    np.fill_diagonal(m, 0.0)
    return m


def _fat_tree(rs, degraded=0.0):
    """4096 GPUs, 2:1 oversubscribed at the core; `degraded`: share of the
    cables at half rate."""
    n = 4096 + 16 * 16 * 16 + 16 * 16 * 8
    bad = np.sort(rs.permutation(n)[:int(degraded * n)]).astype(np.int64)
    return _topology("fat_tree", 512, 2, 50e9, 50e9, int(rs.randint(1 << 31)), pods=16, edges=16, aggs=16, ups=8,
                     degraded=bad, degraded_Bps=25e9)


def _a2a_plan(case, rs):
    p, ops = case["ranks"], []
    for g in range(case["groups"]):
        b, l = divmod(g, 8)
        ranks = np.array([8 * (64 * b + s) + l for s in range(p)])
        after = []
        for ph in range(case.get("phases", 1)):
            m = _zipf(rs, p) if ph % 2 == 0 else m.T.copy()
            ops.append(("a2a", ranks, m, 50e-6 * rs.rand(), after))
            ops.append(("barrier", [len(ops) - 1]))
            after = [len(ops) - 1]
    return [(_fat_tree(rs, 0.1 if case["kind"] == "noalloc" else 0.0), ops)]


def _whatif_plan(case, rs):
    plan = []
    for k in range(case["scenarios"]):
        tp, pp = (4, 8)[k % 2], (4, 8, 16)[k // 2 % 3]
        nic = float(rs.choice([25e9, 50e9, 100e9]))
        n = case["servers"] * 8
        dp = n // (tp * pp)
        topo = _topology("rail", case["servers"], 32, nic, nic, int(rs.randint(1 << 31)),
                         spines=32 // int(rs.choice([1, 2, 4])))
        ids = np.arange(n).reshape(dp, pp, tp)
        ops = [("ring", "aggregated", ids[:, q, t], 4 * GiB, 0.0, []) for t in range(tp) for q in range(pp)]
        a, b = ids[:, :-1, :].ravel(), ids[:, 1:, :].ravel()
        src, dst = np.concatenate([a, b]), np.concatenate([b, a])
        ops.append(("sends", src, dst, np.full(len(src), 128 * MiB), np.zeros(len(src)), None))
        plan.append((topo, ops))
    return plan


def _fattree_plan(case, rs):
    n = 1024 + 1024 + 1024
    topo = _topology("fat_tree", 128, 1, 50e9, 50e9, int(rs.randint(1 << 31)), pods=16, edges=8, aggs=8, ups=8,
                     degraded=np.sort(rs.permutation(n)[:n // 10]).astype(np.int64), degraded_Bps=25e9)
    p = case["ranks"]
    servers = np.arange(p) * 128 // p
    ops = [("ring", "chained", 8 * servers + g, 16 * MiB * p, 0.0, []) for g in range(case["groups"])]
    k = case["background"]
    src = rs.randint(0, 1024, k)
    dst = (src + 1 + rs.randint(0, 1023, k)) % 1024
    ops.append(("sends", src, dst, np.rint(2.0 ** (20 + 6 * rs.rand(k))), 0.02 * rs.rand(k), None))
    return [(topo, ops)]


def _plan(case, seed):
    rs = np.random.RandomState((seed * 2654435761 + 12345) % (1 << 32))
    kind = case["kind"]
    if kind in ("trace", "rollback"):
        return _trace_plan(case, rs)
    make = dict(ring=_ring_plan, step=_step_plan, a2a=_a2a_plan, solve=_a2a_plan, noalloc=_a2a_plan,
                whatif=_whatif_plan, fattree=_fattree_plan)[kind]
    return make(case, rs), None


# -------------------------------------------------------- the framework's calls
_KIND = dict(leaf_spine=ns.TOPO_LEAF_SPINE, rail=ns.TOPO_RAIL, fat_tree=ns.TOPO_FAT_TREE)
_MODE = dict(chained=ns.MODE_CHAINED, flat=ns.MODE_FLAT, aggregated=ns.MODE_AGGREGATED)


def _struct(t):
    s = ns.netsim_topology()
    s.kind, s.servers, s.gpus_per_server, s.servers_per_leaf = _KIND[t["kind"]], t["servers"], t["gpus"], t["per_leaf"]
    s.spines, s.pods, s.edges_per_pod = t["spines"], t["pods"], t["edges"]
    s.aggs_per_pod, s.agg_uplinks = t["aggs"], t["ups"]
    s.nvlink_Bps, s.nic_Bps, s.fabric_Bps, s.ecmp_seed = t["nv"], t["nic"], t["fabric"], t["seed"]
    s.num_degraded, s.degraded_Bps = len(t["degraded"]), t["degraded_Bps"]
    if len(t["degraded"]):
        s.degraded_cables = t["degraded"].ctypes.data_as(ns.ctypes.POINTER(ns.ctypes.c_int64))
    s.fabric_latency_s = s.nvlink_latency_s = t["latency"]
    return s


def _load(plan, opt):
    """A handle with the plan's flows, and the completion flows of every
    operation issued on streams."""
    h = ns.netsim_create_topology([_struct(t) for t, _ in plan], opt)
    done = []
    for s, (_, ops) in enumerate(plan):
        exits, done = [], []
        for op in ops:
            after = []
            if op[0] in ("ring", "a2a"):
                after = np.concatenate([exits[k] for k in op[-1]]) if op[-1] else ()
            if op[0] == "ring":
                ns.netsim_add_ring(h, s, ns.RING_ALLREDUCE, _MODE[op[1]], op[2], op[3], op[4], after)
            elif op[0] == "a2a":
                ns.netsim_add_all_to_all(h, s, op[1], op[2], op[3], after)
            elif op[0] == "barrier":
                d = np.concatenate([exits[k] for k in op[1]])
                ns.netsim_add_flows(h, s, [0.0], [0.0], src=[-1], dst=[-1], dep_off=[0, len(d)], dep_ids=d)
            elif op[0] == "sends":
                kw = {}
                if op[5] is not None:
                    first = ns.netsim_counts(h)[0]
                    kw = dict(dep_off=np.concatenate([[0], np.cumsum([len(x) for x in op[5]])]),
                              dep_ids=np.array([first + j for x in op[5] for j in x], np.int64))
                ns.netsim_add_flows(h, s, op[3], op[4], src=op[1], dst=op[2], **kw)
            elif op[0] == "compute":
                done.append([ns.netsim_stream_compute(h, s, op[1], op[2], [done[k][j] for k, j in op[3]])])
                continue
            elif op[0] == "allreduce" and op[1] == "ring":
                done.append(ns.netsim_stream_ring(h, s, ns.RING_ALLREDUCE, ns.MODE_CHAINED, op[2], op[3], op[4]))
                continue
            elif op[0] == "allreduce":
                done.append(ns.netsim_stream_tree_allreduce(h, s, op[2], op[3], op[4]))
                continue
            else:
                d = ns.netsim_stream_send(h, s, *op[1:])
                done.append([d, ns.netsim_stream_tail(h, s, op[4])])
                continue
            exits.append(ns.netsim_last_exits(h))
    return h, done


class _State:
    """A handle, freed with the state, and what the pass needs beside it."""

    def __init__(self, case, handle=None):
        self.case, self.handle = case, handle

    def __del__(self):
        if self.handle:
            ns.netsim_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    kind = case["kind"]
    plan, moved = _plan(case, seed)
    opt = ns.make_options(exact=case.get("exact", 0), history_mb=case.get("history_mb", 0))
    h, done = _load(plan, opt)
    st = _State(case, h)
    if kind == "rollback":
        st.flow, st.seconds = done[moved][0], plan[0][1][moved][2]
    if kind == "whatif":
        st.scenarios = case["scenarios"]
    if kind == "solve":
        st.ids = np.nonzero(ns.netsim_export_flows(h)["nbytes"] > 0)[0]
    if kind == "noalloc":
        fl, cap = ns.netsim_export_flows(h), ns.netsim_get_links(h, 0)
        routed = fl["nbytes"] > 0
        lens = np.diff(fl["path_off"])[routed]
        used = np.unique(fl["path_link"])
        st.cap = torch.from_numpy(cap[used]).cuda()
        st.poff = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
        st.plink = torch.from_numpy(np.searchsorted(used, fl["path_link"]).astype(np.int32)).cuda()
        st.rates = torch.zeros(int(routed.sum()), dtype=torch.float64, device="cuda")
        st.status = torch.zeros(2, dtype=torch.int64, device="cuda")
    return st


def run(st):
    kind, h = st.case["kind"], st.handle
    if kind == "noalloc":
        ns.netsim_solve_rates_noalloc(0, len(st.cap), st.cap.data_ptr(), len(st.rates), st.poff.data_ptr(),
                                      st.plink.data_ptr(), st.rates.data_ptr(), st.status.data_ptr(),
                                      torch.cuda.current_stream())
        return dict(rates=st.rates, status=st.status)
    if kind == "solve":
        return ns.netsim_solve_once(h, 0, st.ids)
    stream = torch.cuda.current_stream()
    if kind == "rollback":
        ns.netsim_set_limits(h, st.case["step_events"])
        ns.netsim_run(h, stream)
        ns.netsim_update_start(h, st.flow, st.seconds)
        for _ in range(2):
            ns.netsim_advance(h, max_events=st.case["step_events"], stream=stream)
        ns.netsim_advance(h, stream=stream)
        before = ns.netsim_get_finish(h)
        ns.netsim_update_start(h, st.flow, 1.5 * st.seconds)
        ns.netsim_advance(h, stream=stream)
        return dict(before=before, after=ns.netsim_get_finish(h))
    ns.netsim_run(h, stream)
    if kind == "whatif":
        return dict(finish=ns.netsim_get_finish(h), makespan=ns.netsim_get_makespan(h, st.scenarios))
    return ns.netsim_get_finish(h)


def work(case):
    """Bytes: each flow's size, start and dependencies, its path and the links'
    capacities read once, its result written once.  Operations: one division
    per link and three per flow-link pair (count, residual, comparison), as
    if one rate solve sufficed."""
    plan, _ = _plan(case, 0)
    flows = pairs = links = deps = 0
    for topo, ops in plan:
        f = _flows(topo, ops, paths=False)
        flows += len(f["nbytes"])
        pairs += int(f["hops"].sum())
        deps += f["dep_off"][-1]
        links += _num_links(topo)
    if case["kind"] in ("solve", "noalloc"):
        return dict(bytes=8.0 * flows + 4.0 * pairs + 8.0 * links, flops=3.0 * pairs + links)
    return dict(bytes=24.0 * flows + 4.0 * pairs + 8.0 * links + 8.0 * deps, flops=3.0 * pairs + links)


def tolerance(case):
    # exact mode and the solve on device arrays promise the sequential
    # program's arithmetic bit for bit
    if case.get("exact") or case["kind"] == "noalloc":
        return "exact"
    # four times what a change of every capacity by an ulp, or the other
    # order of sums in `exact`, moves the results by
    if case["kind"] == "ring" and case["mode"] == "chained":
        return {"rel": 4e-12, "max": 4e-11}
    if case["kind"] == "a2a":
        return {"rel": 1e-12, "max": 2e-12}
    return {"rel": 2e-14, "max": 1.2e-13}


# ------------------------------------------------------------ plain reference
def _num_links(t):
    g, n = t["gpus"], t["servers"] * t["gpus"]
    cables = n
    if t["kind"] == "fat_tree":
        cables += t["pods"] * t["edges"] * t["aggs"] + t["pods"] * t["aggs"] * t["ups"]
    else:
        leaves = t["servers"] // t["per_leaf"] * (g if t["kind"] == "rail" else 1)
        cables += leaves * t["spines"]
    return t["servers"] * g * (g - 1) + 2 * cables


def _mix(z):
    """SplitMix64's output function."""
    with np.errstate(over="ignore"):
        z = z + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _routes(t, src, dst):
    """Link ids of every pair's route, padded with -1 to six columns."""
    g, n = t["gpus"], t["servers"] * t["gpus"]
    nv = t["servers"] * g * (g - 1)
    s, d = src // g, dst // g
    i, j = src % g, dst % g
    P = np.full((len(src), 6), -1, np.int64)
    if t["kind"] == "rail":
        groups = t["servers"] // t["per_leaf"]
        ls, ld = i * groups + s // t["per_leaf"], j * groups + d // t["per_leaf"]
    else:
        ls, ld = s // t["per_leaf"], d // t["per_leaf"]
    h = _mix(_mix(np.full(len(src), t["seed"], np.uint64)) ^ ((src.astype(np.uint64) << np.uint64(32)) | dst.astype(np.uint64)))
    inside, leaf = s == d, (s != d) & (ls == ld)
    P[inside, 0] = (s * g * (g - 1) + i * (g - 1) + np.where(j < i, j, j - 1))[inside]
    up, down = nv + 2 * src, nv + 2 * dst + 1
    far = ~inside & ~leaf
    P[leaf, 0], P[leaf, 1] = up[leaf], down[leaf]
    P[far, 0] = up[far]
    if t["kind"] != "fat_tree":
        k = (h % np.uint64(t["spines"])).astype(np.int64)
        P[far, 1] = (nv + 2 * (n + ls * t["spines"] + k))[far]
        P[far, 2] = (nv + 2 * (n + ld * t["spines"] + k) + 1)[far]
        P[far, 3] = down[far]
        return P
    E, A, U = t["edges"], t["aggs"], t["ups"]
    a = (h % np.uint64(A)).astype(np.int64)
    u = ((h // np.uint64(A)) % np.uint64(U)).astype(np.int64)
    ps, pd = ls // E, ld // E
    core0 = n + t["pods"] * E * A
    c1, c4 = n + ls * A + a, n + ld * A + a
    same = far & (ps == pd)
    P[same, 1], P[same, 2], P[same, 3] = (nv + 2 * c1)[same], (nv + 2 * c4 + 1)[same], down[same]
    top = far & (ps != pd)
    P[top, 1], P[top, 4], P[top, 5] = (nv + 2 * c1)[top], (nv + 2 * c4 + 1)[top], down[top]
    P[top, 2] = (nv + 2 * (core0 + (ps * A + a) * U + u))[top]
    P[top, 3] = (nv + 2 * (core0 + (pd * A + a) * U + u) + 1)[top]
    return P


def _capacities(t):
    g, n = t["gpus"], t["servers"] * t["gpus"]
    nv = t["servers"] * g * (g - 1)
    c = np.full(_num_links(t), t["fabric"])
    c[:nv], c[nv:nv + 2 * n] = t["nv"], t["nic"]
    for k in t["degraded"]:
        c[nv + 2 * k:nv + 2 * k + 2] = t["degraded_Bps"]
    return c


def _tree(p):
    """Double binary tree: flows (sender, receiver, flows it waits for) in
    order, and the broadcast flows of each rank."""
    level = [0] + [(u & -u).bit_length() - 1 for u in range(1, p + 1)]
    kids, parent = {u: [] for u in range(1, p + 1)}, {}
    for u in range(2, p + 1, 2):
        kids[u].append(u - (1 << (level[u] - 1)))
        for j in range(level[u] - 1, -1, -1):
            if u + (1 << j) <= p:
                kids[u].append(u + (1 << j))
                break
    for u in kids:
        for c in kids[u]:
            parent[c] = u
    root = 1 << (p.bit_length() - 1)
    up = sorted((u for u in kids if u != root), key=lambda u: (level[u], u))
    down = sorted((u for u in kids if u != root), key=lambda u: (-level[u], u))
    flows, of_rank = [], [[] for _ in range(p)]
    for tree in (0, 1):
        def pos(u):
            return u - 1 if tree == 0 else p - u
        r0 = len(flows)
        red = {u: r0 + k for k, u in enumerate(up)}
        bc = {u: r0 + p - 1 + k for k, u in enumerate(down)}
        for c in up:
            flows.append((pos(c), pos(parent[c]), [red[x] for x in kids[c]]))
        for c in down:
            q = parent[c]
            flows.append((pos(q), pos(c), [red[x] for x in kids[q]] if q == root else [bc[q]]))
            of_rank[pos(q)].append(bc[c])
            of_rank[pos(c)].append(bc[c])
    return flows, of_rank


def _flows(topo, ops, paths=True):
    """The flows of one scenario in the order the library numbers them."""
    src, dst, nb, st, deps = [], [], [], [], []

    def add(a, b, n, lag, wait):
        src.append(int(a)), dst.append(int(b)), nb.append(float(n)), st.append(float(lag)), deps.append(list(wait))
        return len(src) - 1

    def ring(mode, ranks, nbytes, lag, after):
        p = len(ranks)
        steps, first = 2 * (p - 1), len(src)
        n = 1 if mode == "aggregated" else steps
        size = nbytes / p * (steps if mode == "aggregated" else 1)
        for k in range(n):
            entry = mode != "chained" or k == 0
            for i in range(p):
                add(ranks[i], ranks[(i + 1) % p], size, lag if entry else 0.0,
                    after if entry else [first + (k - 1) * p + (i - 1) % p])
        e = first + (steps - 1) * p if mode == "chained" else first
        return list(range(e, len(src)))

    exits, done, tail = [], [], {}
    for op in ops:
        if op[0] == "ring":
            exits.append(ring(*op[1:5], [x for k in op[5] for x in exits[k]]))
        elif op[0] == "a2a":
            after = [x for k in op[4] for x in exits[k]]
            exits.append([add(op[1][i], op[1][j], op[2][i, j], op[3], after)
                          for i in range(len(op[1])) for j in range(len(op[1])) if i != j])
        elif op[0] == "sends":
            first = len(src)
            exits.append([add(a, b, n, lag, [first + x for x in op[5][k]] if op[5] else [])
                          for k, (a, b, n, lag) in enumerate(zip(*op[1:5]))])
        elif op[0] == "barrier":
            exits.append([add(-1, -1, 0.0, 0.0, [x for k in op[1] for x in exits[k]])])
        elif op[0] == "compute":
            wait = sorted({done[k][j] for k, j in op[3]} | ({tail[op[1]]} if op[1] in tail else set()))
            tail[op[1]] = add(-1, -1, 0.0, op[2], wait)
            done.append([tail[op[1]]])
        else:
            streams = list(op[3]) if op[0] == "allreduce" else [op[2], op[4]]
            meet = add(-1, -1, 0.0, 0.0, sorted({tail[s] for s in streams if s in tail}))
            if op[0] == "send":
                f = add(op[1], op[3], op[5], 0.0, [meet])
                ends = [[f], [f]]
            elif op[1] == "ring":
                out = ring("chained", op[2], op[4], 0.0, [meet])
                ends = [[out[i], out[i - 1]] for i in range(len(out))]
            else:
                first = len(src)
                rows, of_rank = _tree(len(op[2]))
                for a, b, wait in rows:
                    add(op[2][a], op[2][b], op[4] / 2, 0.0, [first + x for x in wait] or [meet])
                ends = [[first + x for x in r] for r in of_rank]
            ids = [add(-1, -1, 0.0, 0.0, sorted(set(e))) for e in ends]
            tail.update(zip(streams, ids))
            done.append(ids if op[0] == "allreduce" else [ids[0], ids[1]])
    f = dict(nbytes=np.array(nb), start=np.array(st), src=np.array(src), dst=np.array(dst), done=done,
             dep_off=np.concatenate([[0], np.cumsum([len(x) for x in deps])]).astype(np.int64),
             dep_ids=np.array([x for d in deps for x in d], np.int64))
    routed = f["nbytes"] > 0
    P = np.full((len(src), 6), -1, np.int64)
    P[routed] = _routes(topo, f["src"][routed], f["dst"][routed])
    f["hops"] = (P >= 0).sum(1)
    f["path"] = P
    return f


def _fill(cap, P, links):
    """Max-min rates of the flows with paths P (links ids, -1: none): level by
    level, the links of the smallest share give it to their flows.  Only the
    flows of the level's links are looked at."""
    n = len(P)
    L = len(cap)
    pairs = P >= 0
    fl, ll = np.nonzero(pairs)[0], P[pairs]
    order = np.argsort(ll, kind="stable")
    fl, cnt = fl[order], np.bincount(ll, minlength=L)
    off = np.concatenate([[0], np.cumsum(cnt)])
    R, left = cap.copy(), cnt.copy()
    share = np.full(L, INF)
    share[cnt > 0] = R[cnt > 0] / cnt[cnt > 0]
    rate = np.full(n, -1.0)
    todo = n
    while todo:
        s = share.min()
        at = np.nonzero(share <= s * (1 + 1e-12))[0]
        f = np.unique(np.concatenate([fl[off[l]:off[l + 1]] for l in at]))
        f = f[rate[f] < 0]
        rate[f] = s
        todo -= len(f)
        l, k = np.unique(P[f], return_counts=True)
        if l[0] < 0:
            l, k = l[1:], k[1:]
        R[l] -= k * s
        left[l] -= k
        with np.errstate(divide="ignore", invalid="ignore"):
            share[l] = np.where(left[l] > 0, R[l] / left[l], INF)
    return rate


def _rates(cap, P):
    """_fill over the links in use."""
    used, inv = np.unique(P, return_inverse=True)
    inv = inv.reshape(P.shape)
    if used[0] < 0:
        used, inv = used[1:], inv - 1
    return _fill(cap[used], inv, used)


def _simulate(topo, f, base=None):
    """Finish time of every flow: constant rates between events, completions
    and releases processed together at each instant."""
    n = len(f["nbytes"])
    cap, P, nb, start = _capacities(topo), f["path"], f["nbytes"], f["start"]
    hops = f["hops"]
    late = hops * topo["latency"]
    wait = np.diff(f["dep_off"]).copy()
    order = np.argsort(f["dep_ids"], kind="stable")
    owner = np.repeat(np.arange(n), np.diff(f["dep_off"]))[order]
    soff = np.concatenate([[0], np.cumsum(np.bincount(f["dep_ids"], minlength=n))]) if n else np.zeros(1, int)
    finish, ready = np.full(n, np.nan), np.zeros(n)
    pend = np.nonzero(wait == 0)[0]
    rel = start.copy()
    act, rem, rate = np.zeros(0, np.int64), np.zeros(0), np.zeros(0)
    t = 0.0
    while len(act) or len(pend):
        end = t + rem / rate
        tn = min(end.min() if len(act) else INF, rel[pend].min() if len(pend) else INF)
        over = end <= tn * (1 + 1e-12)
        new = act[over]
        finish[new] = tn + late[new]
        rem = (rem - rate * (tn - t))[~over]
        act, changed, t = act[~over], len(new) > 0, tn
        while True:
            for x in new:
                for g in owner[soff[x]:soff[x + 1]]:
                    ready[g] = max(ready[g], finish[x])
            hit = np.concatenate([owner[soff[x]:soff[x + 1]] for x in new]) if len(new) else np.zeros(0, np.int64)
            if len(hit):
                np.subtract.at(wait, hit, 1)
                g = np.unique(hit)
                g = g[wait[g] == 0]
                rel[g] = start[g] + ready[g]
                pend = np.concatenate([pend, g])
            due = pend[rel[pend] <= t]
            if not len(due):
                break
            pend = pend[rel[pend] > t]
            zero = nb[due] == 0
            new, real = due[zero], due[~zero]
            finish[new] = rel[new]
            if len(real):
                act, rem, changed = np.concatenate([act, real]), np.concatenate([rem, nb[real]]), True
            if not len(new):
                break
        if changed and len(act):
            rate = _rates(cap, P[act])
        elif not len(act):
            rate = np.zeros(0)
    return finish


def _seconds(case):
    """A rough estimate of what `exact` takes."""
    p, kind = case.get("ranks", 0), case["kind"]
    if kind == "a2a":
        return 2e-9 * (case["groups"] * p * (p - 1) * case["phases"]) ** 2.5
    if kind == "step":
        return 0.3 + 1e-3 * case["tp_reps"] * 8 * case["dp"] * case["pp"]
    if kind in ("trace", "rollback"):
        return 1e-3 * case["micro"] * case["pp"] * case["dp"] * case["layers"] * case["tp"] * 2
    if kind == "whatif":
        return 1e-3 * case["scenarios"] * case["servers"]
    if kind == "fattree":
        return 2e-4 * case["groups"] * p * p + 5e-3 * case["background"]
    if kind == "ring" and case["mode"] == "chained" and p % 8:
        return 8e-6 * p ** 3
    return 2.0


def exact(case, seed):
    """What run() returns, from the plan alone, in plain numpy; None where that
    takes too long."""
    if _seconds(case) > 20:
        return None
    plan, moved = _plan(case, seed)
    kind = case["kind"]
    if kind in ("solve", "noalloc"):
        topo, ops = plan[0]
        f = _flows(topo, ops)
        r = _rates(_capacities(topo), f["path"][f["nbytes"] > 0])
        return r if kind == "solve" else dict(rates=r, status=None)
    if kind == "whatif":
        fins = [_simulate(t, _flows(t, ops)) for t, ops in plan]
        return dict(finish=np.concatenate(fins), makespan=np.array([x.max() for x in fins]))
    topo, ops = plan[0]
    f = _flows(topo, ops)
    before = _simulate(topo, f)
    if kind != "rollback":
        return before
    k = f["done"][moved][0]
    f["start"][k] *= 1.5
    return dict(before=before, after=_simulate(topo, f))
