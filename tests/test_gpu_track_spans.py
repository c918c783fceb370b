"""Vertices and ambiguity resolution of tracks given directly: events counted
per block of tracks (few and many events a block, tracks in and out of event
order, one and several tracks a thread), and the minima reset in one stream or
for the tracks' keys alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from synth import config as C
from synth import events as E
from tests.test_gpu_vertices import _compare

pytestmark = pytest.mark.gpu

CFG = C.default_config(vtx_pt_min=0.0)


def _hits(n_events, per_event):
    n = n_events * per_event
    f, u = np.zeros(n, np.float32), np.zeros(n, np.uint8)
    off = (np.arange(n_events + 1) * per_event).astype(np.int32)
    return E.Hits(f, f, f, u, np.zeros(n, np.int16), np.arange(n, dtype=np.int32), off)


def _tracks(rng, n, n_hits, precision):
    from paper_2008_13461_amd import _abi as A
    from paper_2008_13461_amd import api
    dt = torch.float64 if precision == A.PT_FIT_F64 else torch.float32
    t = api.Tracks.empty(n, precision, with_cov=True)
    p = rng.normal(size=(n, 5)) * [0.01, 1, 0.1, 0.01, 4.0] + [0.02, 0, 0, 0, 0]
    t.params.copy_(torch.from_numpy(p).to(dt))
    t.cov.zero_()
    t.cov[:, 14] = torch.from_numpy(rng.uniform(1e-6, 4e-4, n)).to(dt).cuda()
    return t, dt


@pytest.mark.parametrize("n,n_events,used,grouped", [(1, 1, 1, True), (256, 300, 300, False), (257, 700, 700, True),
                                                     (5000, 700, 3, False), (5000, 700, 700, False),
                                                     (600_001, 700, 700, True), (600_001, 400, 400, False)])
def test_vertices_of_tracks_in_any_order(n, n_events, used, grouped):
    from paper_2008_13461_amd import _abi as A
    from paper_2008_13461_amd import api
    rng = np.random.Generator(np.random.PCG64(n + n_events))
    h = _hits(n_events, 4)
    ev = rng.choice(np.sort(rng.permutation(n_events)[:used]), n)
    if grouped:
        ev.sort()
    rows = np.full((n, 8), -1, np.int32)
    rows[:, :4] = ev[:, None] * 4 + np.arange(4)
    hits = api.Hits.from_host(h)
    tup = api.Tuplets.from_rows(torch.from_numpy(rows).cuda(), torch.full((n,), 4, dtype=torch.uint8).cuda())
    prec = A.PT_FIT_F32_F64SOLVE
    trk, _ = _tracks(rng, n, h.n_hits, prec)
    cfg, status = A.make_config(CFG), api.new_status()
    vtx = api.Vertices.empty(n, n_events, n)
    ws = api.new_workspace(api.workspace_size(cfg, h.n_hits, n_events, 64, 64, n))
    ws.fill_(0x5A)
    api.find_vertices(hits, cfg, tup, prec, trk, None, None, vtx, status, ws)
    nv = int(vtx.count.item())
    got = {k: getattr(vtx, k)[:nv].cpu().numpy() for k in ("z", "var", "chi2", "ndf", "n_tracks", "sum_pt2")}
    got["event_first"], got["track_vertex"] = vtx.event_first.cpu().numpy(), vtx.track_vertex.cpu().numpy()
    host = dict(hits=rows, n=np.full(n, 4, np.uint8), params=trk.params.cpu().numpy().astype(np.float64),
                cov=trk.cov.cpu().numpy().astype(np.float64))
    assert _compare(h, host, np.ones(n, bool), got, cfg_d=CFG) == nv


@pytest.mark.parametrize("n,cells_cap", [(1, 15), (1, 16 * 4 + 3), (700, 701), (700, 11_199), (700, 11_200), (700, 50_000)])
@pytest.mark.parametrize("double", [False, True])
def test_ambiguities_with_either_reset(n, cells_cap, double):
    from paper_2008_13461_amd import _abi as A
    from paper_2008_13461_amd import api
    rng = np.random.Generator(np.random.PCG64(n + cells_cap))
    h = _hits(1, min(16 * n, 300))
    rows, nh = np.full((n, 8), -1, np.int32), rng.integers(3, 6, n).astype(np.uint8)
    cells = np.full((n, 7), -1, np.int32)
    for i in range(n):
        rows[i, :nh[i]] = rng.choice(h.n_hits, nh[i], replace=False)
        cells[i, :nh[i] - 1] = cells_cap - 1 - rng.integers(0, min(cells_cap, 900), nh[i] - 1)
    prec = A.PT_FIT_F64 if double else A.PT_FIT_F32_F64SOLVE
    tup = api.Tuplets.from_rows(torch.from_numpy(rows).cuda(), torch.from_numpy(nh).cuda())
    tup.cells = torch.from_numpy(cells).cuda()
    trk, dt = _tracks(rng, n, h.n_hits, prec)
    trk.chi2.copy_(torch.from_numpy(np.round(rng.exponential(3.0, n), 2)).to(dt))     # with ties
    if n > 5:
        trk.chi2[3] = float("nan")
    cfg, status = A.make_config(CFG), api.new_status()
    ws = api.new_workspace(api.workspace_size(cfg, h.n_hits, 1, cells_cap, 64, n))
    ws.fill_(0x5A)
    sel, cnt = api.resolve_ambiguities(api.Hits.from_host(h), cfg, api.Cells.empty(cells_cap, h.n_hits), tup, prec, trk,
                                       status, ws)
    keep = O.ambiguity(rows, cells, nh, trk.chi2.cpu().numpy(), trk.params[:, 3].cpu().numpy())
    assert np.array_equal(sel[:int(cnt.item())].cpu().numpy(), np.nonzero(keep)[0])
