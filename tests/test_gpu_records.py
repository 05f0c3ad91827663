"""The memory pass with interval records (graphs whose gap table does not fit
the LDS): the shapes that go wrong in small graphs, with ops of no edges and no
output appended until the table no longer fits, so that both memory passes
meet them.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2608_15762_amd import ss, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ("makespan", "peak", "violation", "slack", "sumfin")
MODES = {"index": 0, "ready": oracle.READY_ORDER, "ports": oracle.LINK_PORTS}


def padded(g, P, n=12_000, seed=0):
    """g with ops appended up to n, and P with devices drawn for them."""
    rng, more = np.random.default_rng(seed), n - g.n_ops
    big = synth.Gmg(**{**g.__dict__, "n_ops": n, "kinds": [],
                       "pred_ptr": np.concatenate([g.pred_ptr, np.full(more, g.pred_ptr[-1])]).astype(np.int32),
                       "op_req": np.concatenate([g.op_req, np.zeros(more)]).astype(np.int32),
                       "dur": np.concatenate([g.dur, rng.integers(1, 4, (more, g.n_class))]).astype(np.int64),
                       "out_bytes": np.concatenate([g.out_bytes, np.zeros(more)]).astype(np.int64)})
    return big, np.concatenate([P, rng.integers(0, g.n_dev, (len(P), more)).astype(np.uint8)], 1)


def check(g, P, mode="index", layout="row", workspace=None):
    dispatch, links = ("ready" if mode == "ready" else "index"), ("ports" if mode == "ports" else "latency")
    ref = oracle.simulate_batch(g, P, dispatch=MODES[mode], n_threads=8)
    h = ss.Gmg(g)
    A = torch.from_numpy(np.ascontiguousarray(P if layout == "row" else P.T)).cuda()
    ws = None
    if workspace is not None:
        lo, hi = ss.workspace_size(h, len(P), layout=layout, dispatch=dispatch, links=links)
        ws = torch.empty(lo + int((hi - lo) * workspace), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    ss.kernel_timing(True)
    out = ss.simulate_batch(h, A, layout=layout, dispatch=dispatch, links=links, workspace=ws)
    torch.cuda.synchronize()
    n, _ = ss.kernel_time(3)
    ss.kernel_timing(False)
    for f in FIELDS:
        a = out[f].cpu().numpy()
        assert np.array_equal(a, ref[f]), (f, np.argwhere(a != ref[f])[:3].tolist())
    assert n > 0  # interval records were written
    return ref


def random_case(seed, n, D, B, **kw):
    kw = dict(dict(n_req=3, n_slices=4, n_link=2, edge_p=0.25, max_span=9, slice_scale=400, cap_scale=20_000), **kw)
    g = synth.random_gmg(seed, n_ops=n, n_dev=D, **kw)
    P = np.random.default_rng(seed).integers(0, D, (B, n)).astype(np.uint8)
    P[0] = 0  # every op on one device
    P[1, n // 2:] = P[1, n // 2]
    return padded(g, P)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("form", [dict(max_outdeg=2), dict(), dict(n_class=2, max_outdeg=2), dict(n_link=3, max_outdeg=2),
                                  dict(n_class=2, n_link=3), dict(n_link=1, max_outdeg=2, max_bytes=1 << 31, bw_max=1 << 26)])
@pytest.mark.parametrize("n,D", [(65, 255), (600, 3), (2049, 33)])
def test_forms(n, D, form, dispatch):
    """The branch-free writer's form and, each alone and together, what takes a
    graph off it: more successors, device classes, link classes."""
    print(f"{n} ops on {D} devices, {form}, {dispatch}", flush=True)
    check(*random_case(n + D, n, D, 21, **form), mode=dispatch)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("layout,workspace", [("op", None), ("row", 0.0), ("row", 0.02), ("op", 0.3)])
def test_chunks(layout, workspace, dispatch):
    """Odd numbers of candidates in chunks of one, of a few and of many."""
    print(f"{layout}, workspace {workspace}, {dispatch}", flush=True)
    g, P = random_case(3, 300, 5, 131 if workspace != 0.0 else 7)
    P[4, 17] = 5  # names an unknown device
    check(g, P, mode=dispatch, layout=layout, workspace=workspace)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("fan,D", [(8, 4), (9, 4), (64, 48), (200, 255)])
def test_many_successors(fan, D, dispatch):
    rng = np.random.default_rng(fan)
    n = 3 * (fan + 2)
    edges = [(0, v) for v in range(1, fan + 1)] + [(fan + 1, v) for v in range(fan + 2, 2 * fan + 2)]
    edges += [(v, v + fan + 2) for v in range(fan + 2, 2 * fan) if v + fan + 2 < n]
    g = synth.make_gmg(D, ["op"] * n, edges, rng.integers(0, 2, n), [[int(x)] for x in rng.integers(1, 90, n)],
                       rng.integers(0, 5000, n), [[(int(rng.integers(0, 300)), synth.TIME_INF)] for _ in range(D)],
                       [20_000] * D, [0, 50], [5_000, 9_000],
                       link_class=rng.integers(0, 3, (D, D)).astype(np.uint8), bw=(50, 10, 7), lat=(0, 3, 1))
    P = rng.integers(0, D, (29, n)).astype(np.uint8)
    P[::4, :fan] %= min(D, 3)
    check(*padded(g, P), mode=dispatch)


@pytest.mark.parametrize("mode", ["index", "ready", "ports"])
@pytest.mark.parametrize("copies", [20, 200, 900])
def test_events_of_one_gap(copies, mode):
    """The copies for every later op of device 0 arrive during one long op on
    it, whose large input is freed at its finish."""
    n = 2 + 2 * copies
    edges = [(0, 1)] + [(2 + i, 2 + copies + i) for i in range(copies)]
    dur = [[2], [100_000]] + [[1 + i % 7] for i in range(copies)] + [[1]] * copies
    out = [1 << 20, 8] + [64 + 8 * (i % 5) for i in range(copies)] + [8] * copies
    g = synth.make_gmg(4, ["op"] * n, edges, [0] * n, dur, out, [[(0, synth.TIME_INF)]] * 4,
                       [1 << 19, 1 << 24, 1 << 24, 1 << 24], [0], [1 << 20], bw=(1000,), lat=(1,))
    P = np.zeros((9, n), np.uint8)
    for c in range(9):
        P[c, 0] = 1 + c % 3
        P[c, 2:2 + copies] = 1 + (np.arange(copies) + c) % 3
    check(*padded(g, P), mode=mode)


@pytest.mark.parametrize("form", [dict(max_outdeg=2), dict(n_class=2)])
@pytest.mark.parametrize("layout,workspace", [("row", None), ("op", None), ("row", 0.2), ("op", 0.5)])
def test_candidates_past_the_limit(layout, workspace, form):
    """A horizon past 32 bits: candidates that use the device whose windows lie
    there are left to the int64 kernels after the record passes."""
    print(f"{layout}, workspace {workspace}, {form}", flush=True)
    D, B = 5, 90
    g, P = random_case(4, 500, D, B, **form)
    last = slice(int(g.slice_ptr[-2]), int(g.slice_ptr[-1]))
    g.slice_begin[last] += 3 << 31
    g.slice_end[last][:-1] += 3 << 31
    P[P == D - 1] = 0
    late = np.arange(B) % 3 == 1
    P[late, 40] = D - 1
    P[6, 2] = D  # names an unknown device
    ref = check(g, P, layout=layout, workspace=workspace)
    assert np.array_equal((ref["makespan"] > 1 << 32) & (ref["violation"] != 4), late)
