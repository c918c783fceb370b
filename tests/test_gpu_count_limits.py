"""Numbers of cells, links and rows beyond 2^31: reported as 2^31 - 1 with the
overflow flag set, the entries below the capacity as in any overflow, and
nothing written outside the buffers."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2008_13461_amd import _abi as A
from paper_2008_13461_amd import api
from synth import config as C
from synth import events as E

pytestmark = pytest.mark.gpu

MOST = 2**31 - 1
GUARD = 1 << 16   # elements on each side of a guarded buffer
MARK = 0x5A


class _Guarded:
    """The buffers of a product, each in the middle of a larger one."""

    def __init__(self, product):
        self.product, self.around = product, []
        for k, t in vars(product).items():
            b = torch.full((t.numel() + 2 * GUARD,), MARK, dtype=t.dtype, device=t.device)
            setattr(product, k, b[GUARD:GUARD + t.numel()].view(t.shape))
            self.around.append(b)

    def untouched(self):
        return all(bool((b[:GUARD] == MARK).all()) and bool((b[-GUARD:] == MARK).all()) for b in self.around)


def _hits(per_layer, seed=1):
    """One event with per_layer[l] hits on barrel layer l, all azimuths and z."""
    rng = np.random.default_rng(seed)
    layer = np.repeat(np.arange(len(per_layer)), per_layer)
    r = np.array([2.9, 6.8, 10.9])[layer]
    phi, z = rng.uniform(-np.pi, np.pi, layer.size), rng.uniform(-20, 20, layer.size)
    i16 = np.zeros(layer.size, np.int16)
    return E.Hits((r * np.cos(phi)).astype(np.float32), (r * np.sin(phi)).astype(np.float32), z.astype(np.float32),
                  layer.astype(np.uint8), i16, i16.astype(np.int32), np.array([0, layer.size], np.int32))


def _flags(status):
    return int(status[A.PT_ST_FLAGS].item())


@pytest.mark.parametrize("fishbone", [0.0, 0.01])
def test_cells_beyond_31_bits(fishbone):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, cap = 50_000, 1000     # 2.5e9 pairs, every one a doublet
    cfg = A.make_config(C.default_config(cut_mask=0, fishbone_theta=fishbone))
    hits = api.Hits.from_host(_hits([n, n]))
    cells, status = api.Cells.empty(cap, 2 * n), api.new_status()
    g = _Guarded(cells)
    ws = api.new_workspace(api.workspace_size(cfg, 2 * n, 1, cap, 16, 16))
    api.build_doublets(hits, cfg, cells, status, ws)
    assert int(cells.count.item()) == MOST
    assert _flags(status) & A.PT_FLAG_CELLS_OVERFLOW
    assert g.untouched()
    inner, outer, _ = (t.cpu().numpy() for t in cells.valid())
    assert len(np.unique(inner)) == 1 and np.all(inner < n)
    assert len(np.unique(outer)) == cap and np.all((outer >= n) & (outer < 2 * n))
    first = np.sort(cells.inner_first[:n].cpu().numpy().astype(np.int64))
    assert np.array_equal(first, np.minimum(np.arange(n) * n, MOST))
    # the truncated cells are a valid input of the next step
    links = api.Links.empty(16, cap)
    gl = _Guarded(links)
    api.link_cells(hits, cfg, cells, links, status, ws)
    assert int(links.count.item()) == 0 and gl.untouched()


@pytest.mark.parametrize("cells_cap", [5_300_000, (1 << 24) + 1])
def test_links_beyond_31_bits(cells_cap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, mid, cap = 1500, 1000, 5000     # 2.25e9 triplets, every one a link
    cfg = A.make_config(C.default_config(cut_mask=0, ca_theta_barrel=2.0, ca_theta_endcap=2.0, ca_rmax_bpix1=1e9,
                                         ca_rmax_other=1e9, min_hits=3))
    h = _hits([n, mid, n])
    hits = api.Hits.from_host(h)
    cells, links, status = api.Cells.empty(cells_cap, h.n_hits), api.Links.empty(cap, cells_cap), api.new_status()
    tup = api.Tuplets.empty(2 * cap)
    ws = api.new_workspace(api.workspace_size(cfg, h.n_hits, 1, cells_cap, cap, 2 * cap))
    api.build_doublets(hits, cfg, cells, status, ws)
    assert _flags(status) == 0
    g = _Guarded(links)
    api.link_cells(hits, cfg, cells, links, status, ws)
    assert int(links.count.item()) == MOST
    assert _flags(status) == A.PT_FLAG_LINKS_OVERFLOW
    assert g.untouched()
    n_cells = int(cells.count.item())
    inner, outer, _ = (t.cpu().numpy() for t in cells.valid())
    joins = (inner < n) & (outer < n + mid)          # ends on a middle hit
    cnt = links.out_count[:n_cells].cpu().numpy()
    assert np.array_equal(cnt, np.where(joins, n, 0))
    assert np.array_equal(links.out_start[:n_cells].cpu().numpy(),
                          np.minimum(np.cumsum(cnt, dtype=np.int64) - cnt, MOST))
    first = cells.inner_first.cpu().numpy()
    want_in = np.repeat(np.flatnonzero(joins)[: cap // n + 1], n)[:cap]
    assert np.array_equal(links.in_cell.cpu().numpy(), want_in)
    assert np.array_equal(links.out_cell.cpu().numpy(), first[outer[want_in]] + np.arange(cap) % n)
    # of the links only those below the capacity are followed: a row for each
    api.find_ntuplets(hits, cfg, cells, links, tup, status, ws)
    assert int(tup.count_raw.item()) == cap
    rows = tup.cells[:cap, :2].cpu().numpy()
    assert np.array_equal(rows[:, 0], want_in) and np.array_equal(rows[:, 1], links.out_cell.cpu().numpy())


@pytest.mark.parametrize("n_roots", [(1 << 19) + 20_000, (1 << 20) + 1])   # past 2^31, and past 2^32
def test_rows_beyond_31_bits(n_roots):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    deg, cap = 16, 10_000     # three levels of 16 cells behind each root: 4096 rows a root
    n_cells = n_roots + 3 * deg
    i32 = dict(dtype=torch.int32, device="cuda")
    cfg_d = C.default_config(min_hits=4)
    cfg = A.make_config(cfg_d)
    hits = api.Hits.from_host(_hits([4, 4, 4]))
    cells, links = api.Cells.empty(n_cells, hits.n_hits), api.Links.empty(deg * (n_roots + 2 * deg), n_cells)
    cells.inner.zero_()
    cells.outer.fill_(1)
    cells.pair.fill_(cfg_d["pairs"].index([2, 3]))
    cells.pair[:n_roots] = cfg_d["pairs"].index([0, 1])
    cells.count.fill_(n_cells)
    links.out_count.fill_(deg)
    links.out_count[-deg:] = 0
    links.out_start.copy_(torch.cumsum(links.out_count, 0) - links.out_count)
    links.count.fill_(links.cap)
    links.has_inner.fill_(1)
    links.in_cell.zero_()
    a = torch.arange(deg, **i32)
    level = torch.cat([torch.zeros(n_roots, **i32), torch.ones(deg, **i32), torch.full((deg,), 2, **i32)])
    links.out_cell.copy_((n_roots + deg * level[:, None] + a).reshape(-1))
    tup, status = api.Tuplets.empty(cap), api.new_status()
    g = _Guarded(tup)
    ws = api.new_workspace(api.workspace_size(cfg, hits.n_hits, 1, n_cells, links.cap, cap))
    api.find_ntuplets(hits, cfg, cells, links, tup, status, ws)
    assert int(tup.count_raw.item()) == MOST
    assert _flags(status) == A.PT_FLAG_TUPLETS_OVERFLOW
    assert g.untouched()
    r = np.arange(cap)
    want = np.full((cap, A.PT_MAX_HITS - 1), -1)
    want[:, 0] = r // deg**3
    for d in range(3):
        want[:, 1 + d] = n_roots + d * deg + r // deg**(2 - d) % deg
    assert np.array_equal(tup.cells.cpu().numpy(), want)
    assert np.all(tup.n.cpu().numpy() == 5)
    assert int(tup.count.item()) == cap and np.array_equal(tup.kept.cpu().numpy(), r)
