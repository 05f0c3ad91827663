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
