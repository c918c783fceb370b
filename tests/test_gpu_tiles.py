"""The device-wide listings (bins, doublets, link starts, roots, rows, kept
rows) at the edges of their tiles of 4096 items, with buffers that are not
16-byte aligned, and with a capacity that takes the listings' many-tile form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2008_13461_amd import _abi as A
from paper_2008_13461_amd import api
from synth import config as C
from synth import events as E

pytestmark = pytest.mark.gpu


def _event(n_hits):
    rng = np.random.Generator(np.random.PCG64(n_hits))
    h = E.make_event(rng, n_vertices=1 + n_hits // 110, fixed_tracks=30, noise_frac=0.2)
    assert h.n_hits >= n_hits
    a = {k: getattr(h, k)[:n_hits] for k in ("x", "y", "z", "layer", "module", "track")}
    return E.Hits(**a, event_offsets=np.array([0, n_hits], np.int32))


def _off(t):
    """The tensor's values and size at an address that is not 16-byte aligned."""
    if t.dim() != 1 or t.numel() < 2:
        return t
    b = torch.zeros(t.numel() + 1, dtype=t.dtype, device=t.device)
    return b[1:]


def _run(h, cells_cap, shifted=False):
    cfg = A.make_config(C.default_config(min_hits=3))
    hits = api.Hits.from_host(h)
    cap = dict(cells_cap=cells_cap, links_cap=cells_cap // 4, tuplets_cap=8 * h.n_hits + 1024)
    cells, links = api.Cells.empty(cells_cap, h.n_hits), api.Links.empty(cap["links_cap"], cells_cap)
    if shifted:
        for p in (cells, links):
            for k, t in vars(p).items():
                setattr(p, k, _off(t))
    tup, status = api.Tuplets.empty(cap["tuplets_cap"]), api.new_status()
    ws = api.new_workspace(api.workspace_size(cfg, h.n_hits, 1, *cap.values()))
    ws.fill_(0x5A)          # nothing may rely on a cleared workspace
    api.build_doublets(hits, cfg, cells, status, ws)
    api.link_cells(hits, cfg, cells, links, status, ws)
    api.find_ntuplets(hits, cfg, cells, links, tup, status, ws)
    n = int(cells.count.item())
    assert int(status[0].item()) & ~A.PT_FLAG_TRUNCATED == 0
    out = [*cells.valid(), *links.valid(), links.out_start[:n], links.out_count[:n], links.has_inner[:n],
           *tup.raw(), tup.kept[: int(tup.count.item())], cells.inner_count]
    return [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("n_hits", [1, 2, 1023, 4095, 4096, 4097, 8193])
def test_listings_at_tile_edges_equal_the_oracle(n_hits):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle as O
    h = _event(n_hits)
    inner, outer, pair, li, lo, start, cnt, _, rows, nh, kept, _ = _run(h, 256 * n_hits + 4096)
    ri, ro, rp = O.doublets_binned(C.default_config(), h.x, h.y, h.z, h.layer)
    key = lambda i, o: np.sort(i.astype(np.int64) << 32 | o)
    assert np.array_equal(key(inner, outer), key(ri, ro))
    # out_start is the exclusive scan of out_count, the links come in cell order
    assert np.array_equal(start, np.cumsum(cnt) - cnt)
    assert np.array_equal(li, np.repeat(np.arange(len(cnt)), cnt))
    # a row is kept when no longer row shares one of its cells: by the rows themselves
    ref = O.reconstruct_event(C.default_config(min_hits=3), h.x, h.y, h.z, h.layer)
    got = {tuple(r[:m]) for r, m in zip(rows[kept].tolist(), nh[kept].tolist())}
    assert got == {tuple(r[:m]) for r, m in zip(ref["hits"].tolist(), ref["n"].tolist())}
    assert np.all(np.diff(kept) > 0)


@pytest.mark.parametrize("n_hits", [1023, 8193])
@pytest.mark.parametrize("cells_cap,shifted", [(None, True), ((1 << 24) + 4097, False), ((1 << 24) + 4097, True)])
def test_listings_do_not_depend_on_capacity_or_alignment(n_hits, cells_cap, shifted):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = _event(n_hits)
    small = 256 * n_hits + 4096
    want = _run(h, small)
    got = _run(h, cells_cap or small, shifted)
    assert all(np.array_equal(a, b) for a, b in zip(want, got))
