"""What the performance of this framework is measured on.

The framework evaluates batches of candidate placements over a Global Mapping
Graph (GMG) snapshot, picks the best one, drives the incremental scheduling
loop around that, and fits the estimators the snapshot's times come from.  The
cases below are those calls as a scheduler makes them, from a 32-op graph with
256 candidates to 50,000 ops on 128 devices with 262,144, with both dispatch
rules, both link models, both placement layouts and each kind of scratch.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2608_15762_amd import ss, synth

GIB = synth.GiB
# "simulate" cases: one batch over one snapshot, then the selection
SIMULATE = dict(kind="simulate", tenants=1, models="8b", ops=32, devices=2, nodes=1, slices=4, clip=False,
                mixed=False, cap_mib=0, candidates=256, recipe="uniform", moves=16, dispatch="index",
                links="latency", layout="row", scratch="pool")


def _simulate(name, **kw):
    case = dict(SIMULATE, name=name)
    case.update(kw)
    return case


def listed():
    return [
        # the smallest call: one 32-op request on two devices, a few hundred candidates
        _simulate("tiny-32op-2dev"),
        # one decode step of an 8B model on two nodes of four devices, every candidate drawn at random
        _simulate("decode-322op-8dev", ops=322, devices=8, nodes=2, slices=16, candidates=65_536),
        # four tenants on four nodes; candidates are the partition placement with a few ops moved, an odd number
        # of them
        _simulate("tenants4-2kop-32dev", tenants=4, models="mix", ops=513, devices=32, nodes=4, slices=64,
                  candidates=100_003, recipe="moved"),
        # eight tenants with little memory left per device, in a workspace that the caller keeps
        _simulate("tenants8-10kop-64dev", tenants=8, ops=1250, devices=64, nodes=8, slices=64, cap_mib=560,
                  candidates=131_072, recipe="moved", moves=8, scratch="workspace"),
        # cluster scale: sixteen tenants on sixteen nodes of eight devices
        _simulate("cluster-50kop-128dev", tenants=16, models="mix", ops=3125, devices=128, nodes=16, slices=256,
                  clip=True, candidates=262_144, recipe="half"),
        # the paper's dispatch rule: the op that is ready first runs next
        _simulate("ready-10kop-64dev", tenants=8, ops=1250, devices=64, nodes=8, slices=64, cap_mib=560,
                  candidates=65_536, recipe="moved", moves=8, dispatch="ready"),
        # transfers that contend for the devices' send and receive ports
        _simulate("ports-2kop-32dev", tenants=4, models="mix", ops=513, devices=32, nodes=4, slices=64,
                  candidates=32_768, recipe="moved", links="ports"),
        # a day's idle windows ahead: times beyond 2^32 microseconds
        _simulate("longhorizon-2kop-32dev", tenants=4, models="mix", ops=513, devices=32, nodes=4, slices=2048,
                  candidates=16_384, recipe="moved"),
        # two generations of accelerators, three kinds of link, and the rotary tables of an instance's first op
        # read by every attention op; placements op by op, as a partitioner that works op by op writes them
        _simulate("mixed-2kop-48dev", tenants=3, models="mix", ops=667, devices=48, nodes=6, slices=64, mixed=True,
                  candidates=32_771, recipe="half", layout="op"),
        # one round of the incremental loop at cluster scale: the snapshot of a running schedule is loaded, and
        # every pre-defined partition of the next 400 ops is simulated on it
        dict(name="round-2kop-128dev", kind="round", tenants=16, models="mix", ops=125, devices=128, nodes=16,
             slices=256, clip=True, batch=400, done=400),
        # the incremental loop from the first round to the last completion
        dict(name="loop-2kop-32dev", kind="loop", tenants=4, models="mix", ops=513, devices=32, nodes=4, slices=64,
             clip=False, cap=150, budget=600),
        # feedback of one interval into the operator estimators, their refit, and predictions from them
        dict(name="estimate-65536x5", kind="estimate", estimators=65_536, features=5, samples=1 << 23,
             queries=1 << 20),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["index"] * 5 + ["ready", "ready", "ports", "ports", "long", "long", "mixed", "mixed", "round",
                                       "round", "loop", "estimate", "estimate"])
    if kind == "estimate":
        features = rng.randint(2, 8)
        estimators = _log(rng, 64, 65_536)
        per = _log(rng, 24, 160)
        return dict(kind="estimate", estimators=estimators, features=features,
                    samples=min(estimators * per, (1 << 25) // features), queries=_log(rng, 1_000, 1 << 20))
    # a node holds 2, 4 or 8 devices
    per_node = rng.choice([2, 4, 8])
    nodes = _log(rng, 1, 128 // per_node)
    devices = per_node * nodes
    tenants = _log(rng, 1, 16)
    models = rng.choice(["8b", "mix"])
    if kind == "round":
        ops = _log(rng, 40, 160)
        n = tenants * ops
        return dict(kind="round", tenants=tenants, models=models, ops=ops, devices=devices, nodes=nodes,
                    slices=rng.choice([64, 256]), clip=True, batch=max(8, n // rng.randint(3, 8)),
                    done=n // rng.randint(3, 8))
    if kind == "loop":
        cap = _log(rng, 60, 300)
        return dict(kind="loop", tenants=min(tenants, 8), models=models, ops=_log(rng, 100, 400), devices=devices,
                    nodes=nodes, slices=64, clip=False, cap=cap, budget=cap * rng.randint(2, 4))
    # op evaluations that take about as long with each rule
    most = {"index": 3e9, "ready": 5e8, "ports": 5e7, "long": 6e7, "mixed": 2e8}[kind]
    ops = max(8, _log(rng, 32, 50_000 if kind == "index" else 12_000) // tenants)
    top = max(65, min(262_144, int(most / (ops * tenants))))
    return dict(SIMULATE, tenants=tenants, models=models, ops=ops, devices=devices, nodes=nodes,
                slices=2048 if kind == "long" else rng.choice([16, 64, 128]), clip=kind != "long",
                mixed=kind == "mixed", cap_mib=rng.choice([0, 560]), candidates=_log(rng, 64, top),
                recipe=rng.choice(["uniform", "moved", "half"]), moves=rng.choice([8, 16]),
                dispatch="ready" if kind == "ready" else "index", links="ports" if kind == "ports" else "latency",
                layout=rng.choice(["row", "row", "op"]), scratch=rng.choice(["pool", "pool", "workspace"]))


# ------------------------------------------------------------------ graphs
@functools.lru_cache(maxsize=4)
def _ops(tenants, models, ops, mixed):
    """The operators of all tenants in one index order: (predecessor offsets,
    predecessors, request, durations, output bytes, edges)."""
    reqs = []
    for t in range(tenants):
        model = ("8b", "1b", "70b")[t % 3] if models == "mix" else "8b"
        kinds, edges = synth.request_graph(model, n_ops=ops)
        if mixed:  # the first op of each instance feeds every attention op of the instance
            first, known = 0, set(edges)
            for v, k in enumerate(kinds):
                if k == "embed":
                    first = v
                elif k == "attn" and (first, v) not in known:
                    edges.append((first, v))
        cost = [synth.op_cost(model, "prefill" if t % 4 == 3 else "decode", k) for k in kinds]
        reqs.append((kinds, edges, [synth.roofline_us(f, m) for f, m, _ in cost], [o for _, _, o in cost]))
    _, edges, req, dur, out = synth._merge_requests(reqs)
    e = np.array(sorted((v, u) for u, v in edges), np.int64).reshape(-1, 2)
    ptr = np.zeros(len(dur) + 1, np.int32)
    ptr[1:] = np.cumsum(np.bincount(e[:, 0], minlength=len(dur)))
    return ptr, e[:, 1].astype(np.int32), np.array(req, np.int32), np.array(dur, np.int64), np.array(out, np.int64)


def _gmg(case, rng):
    """A snapshot whose idle windows, capacities and deadlines are drawn from rng."""
    mixed = case.get("mixed", False)
    ptr, idx, req, dur, out = _ops(case["tenants"], case["models"], case["ops"], mixed)
    D, S, R = case["devices"], case["slices"], case["tenants"]
    dev = np.arange(D)
    node = dev // (D // case["nodes"])
    link = (node[:, None] != node[None, :]).astype(np.uint8)
    bw, lat = ([50_000, 12_500], [0, 0]) if case["nodes"] > 1 else ([50_000], [0])
    cls, w = np.zeros(D, np.int32), dur[:, None]
    if mixed:  # pairs of devices on one board, older accelerators on every other node
        link = link + (dev[:, None] // 2 != dev[None, :] // 2).astype(np.uint8)
        bw, lat = [100_000, 50_000, 12_500], [1, 2, 5]
        cls, w = (node % 2).astype(np.int32), np.stack([dur, dur + (dur * 3 + 4) // 5], 1)
    # idle and busy windows in turn: lognormal, idle 36% of the time
    idle = rng.lognormal(math.log(synth.IDLE_MEDIAN_US), 1.0, (D, S))
    busy = rng.lognormal(math.log(synth.BUSY_MEDIAN_US), 1.0, (D, S))
    if case["clip"]:
        idle, busy = (np.clip(x, synth.CLIP_LO_US, synth.CLIP_HI_US) for x in (idle, busy))
    idle, busy = np.maximum(idle.astype(np.int64), 1), np.maximum(busy.astype(np.int64), 1)
    start = np.where(rng.random(D) < 0.64, (rng.random(D) * busy[:, 0]).astype(np.int64), 0)
    begin = np.zeros((D, S + 1), np.int64)
    begin[:, 1:] = np.cumsum(idle + busy, 1)
    begin += start[:, None]
    end = np.concatenate([begin[:, :S] + idle, np.full((D, 1), synth.TIME_INF, np.int64)], 1)
    cap = np.full(D, case["cap_mib"] << 20, np.int64) if case.get("cap_mib") else \
        288 * GIB - rng.integers(150 * GIB, 250 * GIB, D)
    iso = np.bincount(req, weights=dur, minlength=R).astype(np.int64)
    return synth.Gmg(len(dur), D, w.shape[1], len(bw), R, ptr, idx, req, w, out, cls, link.astype(np.uint8),
                     np.array(bw, np.int64), np.array(lat, np.int64), np.arange(D + 1, dtype=np.int64) * (S + 1),
                     begin.reshape(-1), end.reshape(-1), cap, np.zeros(R, np.int64),
                     iso * rng.integers(1200, 2001, R) // 1000)


def _staged(g, groups):
    """[R][len(groups)] lists of devices -> placements: a request's ops cut into
    contiguous stages of about equal duration, one for each device."""
    out = np.zeros((len(groups[0]), g.n_ops), np.uint8)
    for r in range(g.n_req):
        ops = np.nonzero(g.op_req == r)[0]
        w = g.dur[ops, 0]
        before = np.cumsum(w) - w
        for p, devs in enumerate(groups[r]):
            out[p, ops] = np.asarray(devs, np.uint8)[np.minimum(len(devs) - 1, before * len(devs) // w.sum())]
    return out


def _home(g, case):
    """Every request on its node, a stage on each of the node's devices."""
    per = g.n_dev // case["nodes"]
    return _staged(g, [[range(r % case["nodes"] * per, (r % case["nodes"] + 1) * per)] for r in range(g.n_req)])[0]


def _partitions(g, case):
    """The pre-defined partitions: each node's devices in groups of all, half, ... one."""
    per = g.n_dev // case["nodes"]
    sizes = [per >> s for s in range(per.bit_length())]
    groups = [range(n * per + j * k, n * per + j * k + k) for n in range(case["nodes"]) for k in sizes
              for j in range(per // k)]
    return _staged(g, [groups] * g.n_req)


def _placements(g, case, seed):
    """Candidates on the GPU: uniform, or the home placement with up to `moves`
    ops moved to other devices ("half": every second one of each)."""
    gen = torch.Generator("cuda").manual_seed(seed)
    B, N, D, k = case["candidates"], g.n_ops, g.n_dev, case["moves"]
    P = torch.empty((B, N), dtype=torch.uint8, device="cuda")
    home = torch.from_numpy(_home(g, case)).cuda()
    for b0 in range(0, B, 32_768):
        part = P[b0:b0 + 32_768]
        if case["recipe"] != "moved":
            part.random_(0, D, generator=gen)
        if case["recipe"] != "uniform":
            rows = part[1::2] if case["recipe"] == "half" else part
            n = len(rows)
            at = torch.randint(0, N, (n, k), generator=gen, device="cuda")
            to = torch.randint(0, D, (n, k), generator=gen, device="cuda").to(torch.uint8)
            stay = torch.arange(k, device="cuda") > torch.randint(0, k, (n, 1), generator=gen, device="cuda")
            moved = home.expand(n, N).contiguous()
            moved.scatter_(1, at, torch.where(stay, home[at], to))
            rows.copy_(moved)
    return P.t().contiguous() if case["layout"] == "op" else P


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] == "estimate":
        ptr, x, y, of, q = _samples(case, seed)
        return dict(case=case, ptr=ptr, x=x, y=y, of=of, q=q,
                    est=ss.Estimators(case["estimators"], case["features"]))
    g = _gmg(case, rng)
    if case["kind"] == "loop":
        return dict(case=case, g=g, part=_partitions(g, case), key=int(rng.integers(1 << 62)))
    if case["kind"] == "round":
        return _snapshot(case, g, rng)
    h = ss.Gmg(g)
    opts = dict(layout=case["layout"], dispatch=case["dispatch"], links=case["links"])
    work = None
    if case["scratch"] == "workspace":
        _, size = ss.workspace_size(h, case["candidates"], **opts)
        work = torch.empty(min(size, 24 << 30), dtype=torch.uint8, device="cuda")
    return dict(case=case, g=h, P=_placements(g, case, seed), work=work, opts=opts)


def _snapshot(case, g, rng):
    """A running schedule: the first `done` ops have completed, the next ones
    are issued, the last `batch` ones are about to be, one candidate per
    partition of them."""
    N, done = g.n_ops, case["done"]
    issued = N - min(case["batch"], N - done)
    took = np.maximum(1, np.rint(g.dur[:, 0] * rng.uniform(0.75, 1.25, N))).astype(np.int64)
    when = np.sort(rng.integers(0, 200, N))  # the ops were issued in index order
    fin = np.full(N, -1, np.int64)
    for v in range(done):
        preds = g.pred_idx[g.pred_ptr[v]:g.pred_ptr[v + 1]]
        fin[v] = max(when[v], fin[preds].max(initial=0)) + took[v]
    g.t_now = int(max(fin.max(initial=0), when.max()))
    when[issued:] = g.t_now
    g.done_fin, g.issue_at = fin, when
    rows = _partitions(g, case)
    rows[:, :issued] = _home(g, case)[:issued]
    return dict(case=case, g=g, rows=rows)


def _samples(case, seed):
    """Feedback samples grouped by estimator (some operators have not run yet,
    the others at least 16 times) and queries, on the GPU."""
    E, F, S, M = case["estimators"], case["features"], case["samples"], case["queries"]
    rng = np.random.default_rng(seed)
    p = rng.lognormal(0.0, 0.5, E)
    p[rng.integers(0, E, E // 64)] = 0.0
    n = np.where(p > 0, 16, 0)
    n = n + rng.multinomial(S - n.sum(), p / p.sum())
    gen = torch.Generator("cuda").manual_seed(seed)

    def features(rows):  # products of batched matmul shapes, scaled, and a constant
        s = torch.randint(1, 64, (rows, 4), generator=gen, device="cuda").double()
        b, m, k, c = s.unbind(1)
        cols = [torch.ones_like(b), b * m * k * c / 1e5, b * m * k / 1e3, b * k * c / 1e3, b * m * c / 1e3, m / 10,
                k / 10, c / 10]
        return torch.stack(cols[:F], 1).contiguous()

    x = features(S)
    beta = torch.rand((E, F), generator=gen, device="cuda", dtype=torch.float64) * 4.9 + 0.1
    ids = torch.repeat_interleave(torch.arange(E, device="cuda"), torch.from_numpy(n).cuda(), output_size=S)
    noise = torch.randn(S, generator=gen, device="cuda", dtype=torch.float64) * 0.02 + 1
    y = (x * beta[ids]).sum(1) * noise
    ptr = torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int64)).cuda()
    of = torch.randint(0, E, (M,), generator=gen, device="cuda").to(torch.int32)
    return ptr, x, y, of, features(M)


# ------------------------------------------------------------------ run
def run(state):
    kind = state["case"]["kind"]
    if kind == "estimate":
        state["est"].add(state["ptr"], state["x"], state["y"])
        coef, status = state["est"].solve()
        return dict(coef=coef, status=status, us=ss.est_predict(coef, state["of"], state["q"]))
    if kind == "loop":
        return _loop(state)
    if kind == "round":
        g = ss.Gmg(state["g"])
        out = ss.simulate_batch_resume(g, torch.from_numpy(state["rows"]).cuda())
    else:
        g = state["g"]
        out = ss.simulate_batch(g, state["P"], workspace=state["work"], **state["opts"])
    out["best"] = ss.select_best(g, out["violation"], out["sumfin"])
    return out


def _loop(state):
    """Rounds at the current time until one issues nothing, then the next
    completion, until nothing is left to run."""
    g, part, case = state["g"], state["part"], state["case"]
    loop = ss.Scheduler(g, part, synth.request_priority(g), case["budget"], case["cap"])
    cluster = synth.Executor(g, state["key"])
    now, chosen = 0, []
    while True:
        status, ops, p = loop.round(now)
        while status == ss.SS_ROUND_ISSUED:
            chosen.append(p)
            cluster.issue(ops, part[p, ops].tolist(), now)
            status, ops, p = loop.round(now)
        event = cluster.next_completion()
        if event is None:
            break
        now = event[0]
        loop.complete(event[1], now)
    ops_state, place, issued, done = loop.state()
    return dict(chosen=np.array(chosen, np.int64), state=ops_state, place=place, issued=issued, done=done)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Each placement byte, sample or query read once, each output written
    once; an op's ready time, fit, finish and residency in 16 integer
    operations, a sample's products and sums in two operations each."""
    if case["kind"] == "estimate":
        E, F, S, M = case["estimators"], case["features"], case["samples"], case["queries"]
        stats = 8 * (F * F + F + 1)
        return {"bytes": S * (F + 1) * 8 + (E + 1) * 8 + E * (2 * stats + F * 8 + 4) + M * (F * 8 + 4 + 8),
                "flops": S * F * (F + 3) + E * F * F * F + 2 * M * F}
    N = case["tenants"] * case["ops"]
    if case["kind"] == "simulate":
        B, outputs = case["candidates"], 17 + 8 * case["devices"] + 8 * case["tenants"]
    else:
        per = case["devices"] // case["nodes"]
        B, outputs = case["nodes"] * (2 * per - 1), 17 + 8 * case["tenants"]
        if case["kind"] == "loop":  # every op is in the batch once, and in a snapshot of the budget about four times
            N *= 5
        else:
            outputs += 8 * case["devices"]
    return {"bytes": B * (N + outputs), "flops": 16 * B * N}


def tolerance(case):
    """The simulator and the loop compute in whole numbers.  The estimators
    sum up to a few hundred products of 64-bit numbers in any order and solve
    from them (6e-14 from the sums in plain numpy with five features); a
    prediction is rounded up to a whole microsecond."""
    return {"rel": 1e-12, "differ": 1e-5} if case["kind"] == "estimate" else "exact"


def exact(case, seed):
    """The fits from sums in plain numpy.  The other cases' outputs are whole
    numbers, where every correct implementation gives the same."""
    if case["kind"] != "estimate":
        return None
    E, F = case["estimators"], case["features"]
    ptr, x, y, _, _ = _samples(case, seed)
    ptr, z = ptr.cpu().numpy(), torch.cat([x, y[:, None]], 1).cpu().numpy()
    some = np.nonzero(np.diff(ptr) > 0)[0]
    at = ptr[some]
    gram = np.empty((len(some), F, F + 1))
    for i in range(F):
        for j in range(F + 1):
            gram[:, i, j] = np.add.reduceat(z[:, i] * z[:, j], at)
    coef = np.zeros((E, F))
    coef[some] = np.linalg.solve(gram[:, :, :F], gram[:, :, F:])[:, :, 0]
    return dict(coef=coef, status=None, us=None)
