"""Calls whose scratch is limited (ss_simulate_batch_ws, the fixed array of
ss_simulate_batch_noalloc): what they accept, how large their chunks are, and
their results."""
import numpy as np
import pytest

import oracle
from paper_2608_15762_amd import ss, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ("makespan", "peak", "violation", "slack", "sumfin")
FIXED = 128 << 20  # bytes of the fixed array


def outputs(h, B):
    dev = torch.device("cuda:0")
    return dict(makespan=torch.empty(B, dtype=torch.int64, device=dev),
                violation=torch.empty(B, dtype=torch.uint8, device=dev),
                peak=torch.empty((B, h.n_dev), dtype=torch.int64, device=dev),
                slack=torch.empty((B, h.n_req), dtype=torch.int64, device=dev),
                sumfin=torch.empty(B, dtype=torch.int64, device=dev))


def noalloc(h, P, dispatch="index", links="latency", layout="row"):
    """One call in the fixed array, as host arrays."""
    B, flags = ss._layout(h, P, layout, dispatch, links)
    o = outputs(h, B)
    ss._check(ss.lib().ss_simulate_batch_noalloc(h.handle, ss._ptr(P), B, flags, ss._ptr(o["makespan"]),
                                                 ss._ptr(o["peak"]), ss._ptr(o["violation"]), ss._ptr(o["slack"]),
                                                 ss._ptr(o["sumfin"]), ss._stream_ptr(None)))
    torch.cuda.synchronize()
    return {f: o[f].cpu().numpy() for f in FIELDS}


def same(a, ref, idx=slice(None)):
    for f in FIELDS:
        x, y = a[f][idx], ref[f]
        assert np.array_equal(x, y), (f, np.argwhere(x != y)[:3].tolist())


def test_ready_scratch_of_many_candidates():
    """Ready-time dispatch in chunks of one candidate: no more than a counter
    of four bytes a chunk, so a large batch still fits the fixed array."""
    g = synth.build_gmg(0)
    h = ss.Gmg(g)
    for layout in ("row", "op"):
        lo1, _ = ss.workspace_size(h, 64, dispatch="ready", layout=layout)
        lo2, _ = ss.workspace_size(h, 1 << 20, dispatch="ready", layout=layout)
        assert lo2 - lo1 <= 4 << 20
    B = 200_000
    P = torch.from_numpy(synth.placements(g, 0, 0, B)).cuda()
    a = noalloc(h, P, dispatch="ready")
    idx = np.unique(np.linspace(0, B - 1, 300).astype(np.int64))
    same(a, oracle.simulate_batch(g, P.cpu().numpy()[idx], dispatch=oracle.READY_ORDER, n_threads=8), idx)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("config,ops,index,ready", [(1, 322, 16_384, 16_384), (2, 2052, 4096, 2048),
                                                    (3, 10_000, 512, 512)])
def test_chunks_of_the_fixed_array(config, ops, index, ready, dispatch):
    """A schedule launch lasts about as long for one candidate as for as many
    as the chip holds: the fixed array's chunks are no smaller than those the
    interval records' layout had (2.5 schedule launches' worth of them here)."""
    g = synth.build_gmg(config)
    assert g.n_ops == ops
    h = ss.Gmg(g)
    chunk = index if dispatch == "index" else ready
    B = chunk * 5 // 2
    P = torch.from_numpy(synth.placements(g, config, 0, B)).cuda()
    noalloc(h, P[:64], dispatch=dispatch)
    ss.kernel_timing(True)
    a = noalloc(h, P, dispatch=dispatch)
    n, _ = ss.kernel_time(0)
    ss.kernel_timing(False)
    assert 1 <= n <= 3
    idx = np.unique(np.linspace(0, B - 1, 40).astype(np.int64))
    same(a, oracle.simulate_batch(g, P.cpu().numpy()[idx], n_threads=8,
                                  dispatch=oracle.READY_ORDER if dispatch == "ready" else 0), idx)


@pytest.mark.parametrize("dispatch", ["index", "ready"])
@pytest.mark.parametrize("n,outdeg", [(33, 2), (321, 3), (11_901, 2)])
def test_smallest_workspace_holds_one_candidate(n, outdeg, dispatch):
    """Both memory passes, finish rows padded to whole groups of eight: one
    candidate's rows and records are enough."""
    g = synth.random_gmg(7, n_ops=n, n_dev=3, n_req=2, n_link=2, edge_p=0.15, max_outdeg=outdeg,
                         n_slices=4, slice_scale=400, cap_scale=20_000)
    h = ss.Gmg(g)
    B = 70 if n < 1000 else 9
    P = np.random.default_rng(n).integers(0, 3, (B, n)).astype(np.uint8)
    ref = oracle.simulate_batch(g, P, dispatch=oracle.READY_ORDER if dispatch == "ready" else 0, n_threads=8)
    E = len(g.pred_idx)
    for layout in ("row", "op"):
        A = torch.from_numpy(np.ascontiguousarray(P if layout == "row" else P.T)).cuda()
        lo, hi = ss.workspace_size(h, B, layout=layout, dispatch=dispatch)
        # 64 candidates' finish times alone are 512 bytes an op
        assert lo <= 200 * (n + E) + 16 * 1024
        for size in (lo, lo + (hi - lo) // 100, lo + (hi - lo) // 3, hi - 256):
            out = ss.simulate_batch(h, A, layout=layout, dispatch=dispatch,
                                    workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
            torch.cuda.synchronize()
            same({f: out[f].cpu().numpy() for f in FIELDS}, ref)
    if n == 33 and dispatch == "index":  # what 64 candidates with interval records took
        assert ss.workspace_size(h, 64)[0] <= 23_552


@pytest.mark.parametrize("links", ["latency", "ports"])
@pytest.mark.parametrize("layout", ["row", "op"])
def test_smallest_workspace_of_the_general_kernels(links, layout, monkeypatch):
    """A horizon past 32 bits, and ports on a packed graph: a workspace that
    holds one candidate of the general kernels is enough, for both."""
    g = synth.random_gmg(3, n_ops=700, n_dev=4, n_req=3, n_link=2, edge_p=0.3, max_outdeg=2, n_slices=4,
                         slice_scale=400, cap_scale=20_000)
    if links == "latency":  # the last windows begin past 2^32
        last = np.asarray(g.slice_ptr[1:]) - 1
        first = np.setdiff1d(np.arange(len(g.slice_begin)), last)
        g.slice_begin[last] += 1 << 33
        assert len(first)
    h = ss.Gmg(g)
    P = np.random.default_rng(1).integers(0, 4, (70, g.n_ops)).astype(np.uint8)
    ref = oracle.simulate_batch(g, P, dispatch=oracle.LINK_PORTS if links == "ports" else 0, n_threads=8)
    A = torch.from_numpy(np.ascontiguousarray(P if layout == "row" else P.T)).cuda()
    lo, hi = ss.workspace_size(h, len(P), layout=layout, links=links)
    monkeypatch.setenv("SS_PATH", "generic")
    general, _ = ss.workspace_size(h, len(P), layout=layout, links=links)
    monkeypatch.delenv("SS_PATH")
    assert lo <= general
    for size in (lo, lo + 4096, (lo + hi) // 2, hi):
        out = ss.simulate_batch(h, A, layout=layout, links=links,
                                workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        same({f: out[f].cpu().numpy() for f in FIELDS}, ref)
    with pytest.raises(ss.SSError):
        ss.simulate_batch(h, A, layout=layout, links=links,
                          workspace=torch.empty(lo - 256, dtype=torch.uint8, device="cuda"))


def far_graph(n=257, D=5, seed=11, far=3 << 31, **kw):
    """A graph whose last device is idle from `far` on only (past a 32-bit
    horizon): a candidate that uses it passes the limit."""
    g = synth.random_gmg(seed, n_ops=n, n_dev=D, **dict(dict(n_req=3, n_link=2, edge_p=0.3, max_outdeg=2, n_slices=4,
                                                             slice_scale=400, cap_scale=20_000), **kw))
    last = slice(int(g.slice_ptr[-2]), int(g.slice_ptr[-1]))
    g.slice_begin[last] += far
    g.slice_end[last][:-1] += far
    return g


@pytest.mark.parametrize("scratch", ["pool", "small", "middle"])
@pytest.mark.parametrize("layout", ["row", "op"])
@pytest.mark.parametrize("B,share", [(300, 0.5), (17_000, 0.03), (17_000, 0.49), (17_000, 0.99), (40_001, 0.6)])
def test_candidates_past_the_limit(B, share, layout, scratch):
    """Candidates left to the int64 kernels: few, up to and past the number
    from which a lane schedules each, in one chunk and in several."""
    g = far_graph()
    h = ss.Gmg(g)
    rng = np.random.default_rng(B)
    P = rng.integers(0, g.n_dev - 1, (B, g.n_ops)).astype(np.uint8)
    late = rng.random(B) < share
    P[late, rng.integers(0, g.n_ops, int(late.sum()))] = g.n_dev - 1
    P[B // 2, 5] = g.n_dev  # names an unknown device
    ref = oracle.simulate_batch(g, P, n_threads=8)
    assert np.array_equal((ref["makespan"] > 1 << 32) & (ref["violation"] != 4), late & (np.arange(B) != B // 2))
    A = torch.from_numpy(np.ascontiguousarray(P if layout == "row" else P.T)).cuda()
    lo, hi = ss.workspace_size(h, B, layout=layout)
    size = {"pool": None, "small": hi // 20, "middle": hi // 3}[scratch]
    ws = None if size is None else torch.empty(max(lo, size), dtype=torch.uint8, device="cuda")
    out = ss.simulate_batch(h, A, layout=layout, workspace=ws)
    torch.cuda.synchronize()
    same({f: out[f].cpu().numpy() for f in FIELDS}, ref)


def test_scratch_past_the_limit():
    """The int64 kernels reuse the 32-bit ones' scratch: about four bytes a
    candidate more than the same graph without far windows takes (while a wave
    schedules each; a lane each keeps the requests' completions too)."""
    near, far = ss.Gmg(far_graph(far=0)), ss.Gmg(far_graph())
    B = 8_192
    assert ss.workspace_size(far, B)[1] <= ss.workspace_size(near, B)[1] + 8 * B + 4096
