"""The general (int64) kernels where their variants meet: the schedule with a
wave per candidate and with a lane per candidate (up to 16,384 candidates, 8,192
with fewer than four requests or devices, 7,168 on one device, and 512 requests,
and beyond), its 64-op chunks, inputs from the same chunk, and
the memory pass's three ways to hold a device's endpoints (a wave's share of
the LDS, all of it, the global buffer).  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2608_15762_amd import ss, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ("makespan", "peak", "violation", "slack", "sumfin")


@pytest.fixture(autouse=True)
def general(monkeypatch):
    monkeypatch.setenv("SS_PATH", "generic")


def check(g, P, run=ss.simulate_batch, ref=None):
    ref = oracle.simulate_batch(g, P, n_threads=8) if ref is None else ref
    out = run(ss.Gmg(g), torch.from_numpy(P).cuda())
    torch.cuda.synchronize()
    for f in FIELDS:
        a = out[f].cpu().numpy()
        assert np.array_equal(a, ref[f]), (f, np.argwhere(a != ref[f])[:3].tolist())


def graph(seed, n, D=5, **kw):
    return synth.random_gmg(seed, n_ops=n, n_dev=D, **dict(dict(n_req=3, n_slices=6, n_class=2, n_link=3, rel_max=20,
                                                                cap_scale=6000), **kw))


def batch(g, B, seed=0):
    P = np.random.default_rng(seed).integers(0, g.n_dev, (B, g.n_ops)).astype(np.uint8)
    P[0] = g.n_dev - 1
    P[-1, -1] = g.n_dev  # names an unknown device
    return P


@pytest.mark.parametrize("B,n_req", [(1, 3), (8192, 3), (8193, 3), (16384, 3), (16384, 4), (16385, 4)])
@pytest.mark.parametrize("snapshot", [False, True])
def test_batch_sizes(B, n_req, snapshot):
    print(f"{B} candidates, {n_req} requests, snapshot {snapshot}", flush=True)
    g = graph(3, 130, n_req=n_req)
    check(synth.random_snapshot(g, 5, done_p=0.5) if snapshot else g, batch(g, B) if B > 1 else batch(g, 2)[:1])


@pytest.mark.parametrize("B", [40, 8195, 16400])
def test_resumed(B):
    """Candidates resumed after a prefix that ends inside a chunk."""
    print(f"{B} candidates resumed", flush=True)
    g = graph(4, 150)
    P = batch(g, B)
    P[:, :71] = P[1, :71]
    k = synth.Gmg(**{**g.__dict__, "n_ops": 71, "pred_ptr": g.pred_ptr[:72].copy(),
                     "pred_idx": g.pred_idx[:g.pred_ptr[71]].copy(), "op_req": g.op_req[:71].copy(),
                     "dur": g.dur[:71].copy(), "out_bytes": g.out_bytes[:71].copy()})
    state = ss.State()
    ss.state_capture(ss.Gmg(k), torch.from_numpy(P[1, :71].copy()).cuda(), state)
    check(g, P, run=lambda h, p: ss.simulate_batch_resume(h, p, start=state))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129])
@pytest.mark.parametrize("edge_p,max_span", [(0.2, 3), (0.7, 12), (0.3, 100)])
def test_chunks(n, edge_p, max_span):
    g = graph(n, n, edge_p=edge_p, max_span=max_span)
    check(g, batch(g, 33))
    check(synth.random_snapshot(g, n, done_p=0.6), batch(g, 33))


@pytest.mark.parametrize("n_req", [512, 513])
def test_many_requests(n_req):
    g = graph(9, 700, n_req=n_req)
    check(g, batch(g, 20))


@pytest.mark.parametrize("n,D", [(129, 1), (300, 2), (3000, 2), (5000, 1), (2600, 255)])
def test_endpoints(n, D):
    """About three to four endpoints an op: 512 on a device are a wave's
    share, 8,192 the workgroup's."""
    print(f"{n} ops on {D} devices", flush=True)
    g = graph(11, n, D=D, edge_p=0.2, cap_scale=400_000)
    check(g, np.random.default_rng(n).integers(0, D, (4, n)).astype(np.uint8))
    P = np.zeros((3, n), np.uint8)
    P[1, n // 2:] = D - 1
    P[2, ::3] = D - 1
    check(g, P)


@pytest.mark.parametrize("B", [256, 257, 513])  # sixteen, eight and four waves to a candidate
@pytest.mark.parametrize("n,D", [(61, 1), (128, 1), (300, 1), (500, 1), (300, 3), (700, 3), (2000, 3), (700, 9)])
def test_team_sizes(n, D, B):
    """Workgroups of every size the memory pass has, with devices whose
    endpoints fit a wave's share of its LDS, all of it, or the global buffer:
    a third of the candidates on one device whole."""
    print(f"{B} candidates of {n} ops on {D} devices", flush=True)
    g = graph(12, n, D=D, edge_p=0.2, cap_scale=100_000)
    P = batch(g, B)
    P[::3] = D - 1
    check(g, P)


@pytest.mark.parametrize("B", [7168, 7169])
def test_one_device(B):
    g = graph(13, 70, D=1)
    check(g, batch(g, B))
