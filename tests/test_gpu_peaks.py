"""The memory pass whose gap table lies in LDS, where it can go wrong: sizes
around its chunks, its waves and the largest table a workgroup holds, one
device with every op, ops with many successors, and more events in one gap
than the LDS list holds.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2608_15762_amd import ss, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ("makespan", "peak", "violation", "slack", "sumfin")


def check(g, P, dispatch="index", links="latency"):
    mode = {"ready": oracle.READY_ORDER, "ports": oracle.LINK_PORTS}.get(dispatch if links == "latency" else links, 0)
    ref = oracle.simulate_batch(g, P, dispatch=mode, n_threads=8)
    out = ss.simulate_batch(ss.Gmg(g), torch.from_numpy(P).cuda(), dispatch=dispatch, links=links)
    torch.cuda.synchronize()
    for f in FIELDS:
        a = out[f].cpu().numpy()
        assert np.array_equal(a, ref[f]), (f, np.argwhere(a != ref[f])[:3].tolist())


def random_case(seed, n, D, B, **kw):
    kw = dict(dict(n_req=3, n_slices=4, n_link=2, edge_p=0.25, max_span=9, slice_scale=400, cap_scale=20_000), **kw)
    g = synth.random_gmg(seed, n_ops=n, n_dev=D, **kw)
    P = np.random.default_rng(seed).integers(0, D, (B, n)).astype(np.uint8)
    P[0] = 0  # every op on one device
    P[1, n // 2:] = P[1, n // 2]
    return g, P


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("outdeg", [2, None])
@pytest.mark.parametrize("n,D", [(1, 1), (63, 2), (64, 255), (65, 3), (127, 128), (129, 5), (513, 64), (1100, 7),
                                 (2049, 33)])
def test_sizes(n, D, outdeg, dispatch):
    print(f"{n} ops on {D} devices, out-degree {outdeg}, {dispatch}", flush=True)
    check(*random_case(n + D, n, D, 37, max_outdeg=outdeg), dispatch=dispatch)


def in_lds(g, P, dispatch="index"):
    """Whether the memory pass of a call ran in LDS (no interval records)."""
    h, A = ss.Gmg(g), torch.from_numpy(P).cuda()
    torch.cuda.synchronize()
    ss.kernel_timing(True)
    ss.simulate_batch(h, A, dispatch=dispatch)
    torch.cuda.synchronize()
    n, _ = ss.kernel_time(3)
    ss.kernel_timing(False)
    return n == 0


@pytest.mark.parametrize("max_bytes", [1000, 1 << 31])  # 32- and 64-bit byte sums
@pytest.mark.parametrize("step", [-600, -1, 0, 1, 600])
def test_largest_table(step, max_bytes):
    """12 (20 with 64-bit sums) bytes an entry, two an op of event list: 11,689
    (7,433) ops on three devices fill 160 KB; both sides of it."""
    n = (11_689 if max_bytes == 1000 else 7_433) + step
    print(f"{n} ops, sizes up to {max_bytes}", flush=True)
    g, P = random_case(5, n, 3, 6, max_bytes=max_bytes, max_outdeg=2, edge_p=0.1, cap_scale=max_bytes * 100)
    check(g, P)
    assert in_lds(g, P) == (step <= 0)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("D,max_bytes,last", [(3, 1000, 11_685), (128, 1000, 11_256), (255, 1000, 10_821),
                                              (128, 1 << 31, 7_064)])
@pytest.mark.parametrize("step", [-90, 0, 1, 40])
def test_largest_table_with_wide_successors(step, D, max_bytes, last, dispatch):
    """With device arrays of 12 bytes a device for each wave beside the table:
    the last size that leaves room for two waves, and one wave's beyond."""
    n = last + step
    print(f"{n} ops on {D} devices, sizes up to {max_bytes}, {dispatch}", flush=True)
    # (links fast enough for the horizon to fit 32 bits)
    g, P = random_case(6, n, D, 5, max_bytes=max_bytes, bw_max=max_bytes // 20, edge_p=0.2, n_link=3, n_class=2,
                       cap_scale=max_bytes * 100)
    assert ss.time_bits(ss.Gmg(g), dispatch=dispatch) == 32
    check(g, P, dispatch=dispatch)
    assert in_lds(g, P, dispatch) == (step <= 0)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("fan,D", [(8, 4), (9, 4), (64, 48), (200, 255)])
def test_many_successors(fan, D, dispatch):
    """Ops with `fan` consumers, beside ops with few."""
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
    check(g, P, dispatch=dispatch)


@pytest.mark.parametrize("links", ["latency", "ports"])
@pytest.mark.parametrize("copies", [20, 200, 900])
def test_events_of_one_gap(copies, links):
    """A long op on device 0 during which the copies for every later op of the
    device arrive, and whose large input is freed at its finish: all in one
    gap whose bound exceeds every exact value (the list holds 64 events, or
    one per eight ops)."""
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
    check(g, P, links=links)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
def test_times_past_2_31_with_short_slices(dispatch):
    """Finite slices that end early (so the slice lookup has buckets of 1 us)
    and finishes between 2^31 and 2^32."""
    n = 5
    g = synth.make_gmg(2, ["op"] * n, [(0, 1), (1, 2), (2, 3), (3, 4)], [0] * n, [[820_000_000]] * n, [100] * n,
                       [[(0, 40), (90, synth.TIME_INF)], [(7, synth.TIME_INF)]], [150, 1000], [0], [1 << 40])
    check(g, np.array([[0] * n, [1] * n, [0, 1, 0, 1, 0], [0, 0, 1, 1, 1]], np.uint8), dispatch=dispatch)


@pytest.mark.parametrize("outdeg,n_class", [(2, 1), (None, 2)])
@pytest.mark.parametrize("ahead", [0.2, 0.55, 0.9, 1.0])
def test_horizon_past_32_bits(ahead, outdeg, n_class):
    """Idle windows beyond 2^32 us: candidates whose times stay below the
    32-bit limit, pass it at the last ops, or pass it everywhere (`ahead` of
    the devices' short windows end near 2^32), alone and mixed in a batch."""
    n, D = 150, 4
    print(f"windows up to {ahead} of 2^32", flush=True)
    g = synth.random_gmg(8, n_ops=n, n_dev=D, n_req=3, n_class=n_class, n_link=2, max_outdeg=outdeg, edge_p=0.2,
                         open_only=True, cap_scale=9000)
    rng = np.random.default_rng(int(ahead * 100))
    begin, end, ptr = [], [], [0]
    for d in range(D):  # windows that hold a few ops each, then a gap, up to well past 2^32
        t = 10 * d
        step = max(200, int(ahead * (1 << 32) / 40)) if d % 2 else 200
        while t < 3 << 31:
            w = int(rng.integers(40, 120))
            begin.append(t)
            end.append(t + w)
            t += w + step + int(rng.integers(0, 50))
            if len(begin) - ptr[-1] > 60:
                step = 1 << 30
        begin.append(t)
        end.append(synth.TIME_INF)
        ptr.append(len(begin))
    g.slice_ptr, g.slice_begin, g.slice_end = (np.array(x, np.int64) for x in (ptr, begin, end))
    P = rng.integers(0, D, (61, n)).astype(np.uint8)
    P[::3] = P[::3] // 2 * 2  # only devices with windows close together
    P[5] = 0
    P[6] = 1
    P[7, -1] = D
    h = ss.Gmg(g)
    assert ss.time_bits(h) == 64
    ref = oracle.simulate_batch(g, P, n_threads=8)
    late = (ref["makespan"] >= 1 << 32) & (ref["violation"] != 4)
    print(f"{int(late.sum())} of {len(P)} candidates pass 2^32", flush=True)
    # a horizon past 2^32 without its 32-bit tables would run no LDS memory pass
    # beside the int64 one: two memory kernels, the second for marked candidates
    assert 0 < late.sum() < len(P) - 1
    check(g, P)
    A = torch.from_numpy(P).cuda()
    torch.cuda.synchronize()
    ss.kernel_timing(True)
    ss.simulate_batch(h, A)
    torch.cuda.synchronize()
    n, _ = ss.kernel_time(1)
    ss.kernel_timing(False)
    assert n == 2


@pytest.mark.parametrize("D,fan", [(3, 127), (40, 130), (255, 600), (64, 2000)])
def test_many_pending_transfers(D, fan):
    """Producers of equal length on all devices but one, each with a consumer
    on device 0 whose receive port takes the transfers one by one: more than
    the 128 pending transfers held in LDS, every input count up to five."""
    rng = np.random.default_rng(fan)
    n = fan + fan // 3
    edges, at = [], 0
    for v in range(fan, n):
        for u in range(at, min(fan, at + 1 + v % 5)):
            edges.append((u, v))
        at += 1 + v % 5
    g = synth.make_gmg(D, ["op"] * n, edges, rng.integers(0, 3, n), [[3]] * fan + [[int(x)] for x in rng.integers(1, 9, n - fan)],
                       rng.integers(0, 900, n), [[(int(rng.integers(0, 2)), synth.TIME_INF)] for _ in range(D)],
                       [20_000] * D, [0, 2, 9], [5_000, 9_000, 0], link_class=rng.integers(0, 2, (D, D)).astype(np.uint8),
                       bw=(40, 9), lat=(0, 2))
    P = np.zeros((23, n), np.uint8)
    for c in range(23):
        P[c, :fan] = 1 + (np.arange(fan) * (c + 1)) % (D - 1)
        P[c, fan:] = rng.integers(0, 2 if c % 2 else 1, n - fan)
    P[4, 3] = D if D < 255 else 255  # names an unknown device
    check(g, P, links="ports")
    check(g, P)


@pytest.mark.parametrize("layout", ["row", "op"])
@pytest.mark.parametrize("width", [2, 4, 5, 8, 10, 11, 16, 31, 33, 64])
def test_ready_widths(width, layout):
    """`width` ops ready at once (chains out of a binary tree, some joined
    again): each slot count of the ready-time lanes, and more than they hold."""
    rng = np.random.default_rng(width)
    edges, leaves, n = [], [0], 1
    while len(leaves) < width:  # split the earliest leaf in two
        v = leaves.pop(0)
        edges += [(v, n), (v, n + 1)]
        leaves += [n, n + 1]
        n += 2
    for _ in range(6):  # chains, now and then two joined into one and split again
        nxt = []
        for i, v in enumerate(leaves):
            edges.append((v, n))
            nxt.append(n)
            n += 1
        leaves = nxt
        if len(leaves) > 2:
            edges += [(leaves[0], n), (leaves[1], n), (n, n + 1), (n, n + 2)]
            leaves = leaves[2:] + [n + 1, n + 2]
            n += 3
    D, B = 5, 101
    g = synth.make_gmg(D, ["op"] * n, edges, rng.integers(0, 3, n), [[int(x), int(x) + 2] for x in rng.integers(1, 30, n)],
                       rng.integers(0, 900, n), [[(3 * d, 40 + 6 * d), (70 + d, synth.TIME_INF)] for d in range(D)],
                       [4_000] * D, [0, 11, 5], [600, 900, 300], link_class=rng.integers(0, 2, (D, D)).astype(np.uint8),
                       bw=(40, 9), lat=(1, 4), dev_class=[d % 2 for d in range(D)])
    P = rng.integers(0, D, (B, n)).astype(np.uint8)
    P[3], P[9, -1] = 1, D
    ref = oracle.simulate_batch(g, P, dispatch=oracle.READY_ORDER, n_threads=8)
    A = torch.from_numpy(np.ascontiguousarray(P if layout == "row" else P.T)).cuda()
    out = ss.simulate_batch(ss.Gmg(g), A, dispatch="ready", layout=layout)
    torch.cuda.synchronize()
    for f in FIELDS:
        assert np.array_equal(out[f].cpu().numpy(), ref[f]), f
