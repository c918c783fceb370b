"""The fit's lists per number of hits at the edges of a wavefront's 64 tracks,
with the capacities on both sides of the one where a kernel per range of
numbers takes the place of the one that fits them all."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from synth import config as C
from synth import events as E
from tests.helpers import param_rel_err

pytestmark = pytest.mark.gpu

CFG = C.default_config()
RADII = [2.9, 4.4, 6.8, 8.6, 10.9, 13.2, 16.0, 18.2]
MERGED = 131072      # the largest capacity of the one kernel
GRADS = 1 << 21      # and of the adjoint's


@pytest.mark.parametrize("per_n", [{3: 63, 4: 64, 5: 65, 6: 1, 8: 130, 2: 3, 9: 2}, {7: 1}, {2: 70}, {4: 129, 7: 64}])
@pytest.mark.parametrize("cap", [MERGED, MERGED + 1, GRADS + 1])
@pytest.mark.parametrize("precision_name,tol,gtol", [("PT_FIT_F64", 1e-9, 1e-8),
                                                     ("PT_FIT_F32_F64SOLVE", 1e-4, 1e-3)])
def test_lists_of_mixed_lengths(per_n, cap, precision_name, tol, gtol):
    from paper_2008_13461_amd import _abi as A
    from paper_2008_13461_amd import api
    precision = getattr(A, precision_name)
    double = precision == A.PT_FIT_F64
    nh = np.concatenate([np.full(c, n, np.uint8) for n, c in per_n.items()])
    nh = np.random.Generator(np.random.PCG64(7)).permutation(nh)
    n = len(nh)
    ts = E.cylinder_tracks(5, n, RADII, dtype=np.float64 if double else np.float32)
    h, off, g = ts.hits, E.module_offsets(), E.cotangents(3, n)
    good = (nh >= 3) & (nh <= 8)
    g[0][~good] = g[1][~good] = 0.0

    tup = api.Tuplets.empty(cap)
    tup.kept = None
    tup.hits[:n] = torch.from_numpy(ts.tuplets).cuda()
    tup.n[:n] = torch.from_numpy(nh).cuda()
    tup.count.fill_(n)
    cfg = A.make_config(CFG)
    hits, tracks, status = api.Hits.from_host(h), api.Tracks.empty(cap, precision), api.new_status()
    ws = api.new_workspace(api.workspace_size(cfg, h.n_hits, 1, 0, 0, cap))
    ws.fill_(0x5A)
    dt = torch.float64 if double else torch.float32
    offs = torch.from_numpy(off).cuda()
    api.fit_broken_line(hits, cfg, tup, offs, precision, tracks, status, ws)
    assert int(status[A.PT_ST_FIT_FAILED].item()) == int((~good).sum())
    gp, gc = torch.zeros((cap, 5), dtype=dt, device="cuda"), torch.zeros((cap,) + g[1].shape[1:], dtype=dt, device="cuda")
    gp[:n], gc[:n] = torch.from_numpy(g[0]).cuda().to(dt), torch.from_numpy(g[1]).cuda().to(dt)
    gh = torch.zeros((h.n_hits, 3), dtype=dt, device="cuda")
    go = torch.zeros((C.N_MODULES, 3), dtype=torch.float64, device="cuda")
    api.fit_broken_line_bwd(hits, cfg, tup, offs, precision, gp, gc, gh, go, status, ws)
    st = tracks.status[:n].cpu().numpy()
    assert np.all(st[good] & 5 == 0) and np.all(st[~good] & A.PT_FIT_ST_FAILED)
    assert torch.isnan(tracks.params[:n].cpu()[torch.from_numpy(~good)]).all()
    if not good.any():
        assert not gh.any() and not go.any()
        return
    args = (ts.tuplets[good], nh[good], h.x, h.y, h.z, h.layer, h.module, off)
    ref, chi2, _ = O.fit(CFG, *args)
    assert param_rel_err(tracks.params[:n].cpu().numpy().astype(np.float64)[good], ref).max() <= tol
    cerr = np.abs(tracks.chi2[:n].cpu().numpy().astype(np.float64)[good] - chi2) / np.maximum(np.abs(chi2), 1.0)
    assert cerr.max() <= (tol if double else 1e-3)
    gh_ref, go_ref = O.fit_grad(CFG, *args, g[0][good], g[1][good])
    got = gh.cpu().numpy().astype(np.float64)
    rows = ts.tuplets[good]
    num, den = (np.linalg.norm(a[rows], axis=(1, 2)) for a in (got - gh_ref, gh_ref))
    assert np.all(num <= gtol * den)
    assert np.abs(go.cpu().numpy() - go_ref).max() <= gtol * np.abs(go_ref).max()


def test_more_wavefronts_than_a_few_rounds():
    """Past 8192 portions of 64 tracks the order of the portions turns round: 54
    copies of 20 000 tracks of 3 to 8 hits give the oracle's fits of one."""
    from paper_2008_13461_amd import _abi as A
    from paper_2008_13461_amd import api
    n, copies = 20_000, 54     # half of them have 4 to 6 hits: 8438 portions
    ts = E.cylinder_tracks(6, n, RADII)
    nh = np.random.Generator(np.random.PCG64(8)).integers(3, 9, n).astype(np.uint8)
    h = ts.hits
    rows = torch.from_numpy(ts.tuplets).cuda().repeat(copies, 1)
    tup = api.Tuplets.from_rows(rows, torch.from_numpy(nh).cuda().repeat(copies))
    cfg = A.make_config(CFG)
    tracks, status = api.Tracks.empty(n * copies, A.PT_FIT_F32_F64SOLVE), api.new_status()
    ws = api.new_workspace(api.workspace_size(cfg, h.n_hits, 1, 0, 0, n * copies))
    api.fit_broken_line(api.Hits.from_host(h), cfg, tup, None, A.PT_FIT_F32_F64SOLVE, tracks, status, ws)
    ref, _, _ = O.fit(CFG, ts.tuplets, nh, h.x, h.y, h.z, h.layer)
    got = tracks.params.view(copies, n, 5).cpu().numpy().astype(np.float64)
    for c in (0, 1, copies - 1):
        assert param_rel_err(got[c], ref).max() <= 1e-4
    assert np.array_equal(got, np.broadcast_to(got[0], got.shape))
