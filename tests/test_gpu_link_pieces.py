"""The link search of hits at the edges of what is staged at once (192 places,
pieces of 96 out-cells beyond), of the flags kept on the chip (1024
out-cells), of a wavefront's 64 in-cells, with out-cells that have no
direction, and with cuts too wide for direction bins."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from synth import config as C
from synth import events as E
from tests.helpers import doublet_set, link_set
from tests.test_gpu_edge import _doublets_and_links, _star_event

pytestmark = pytest.mark.gpu


def _event(n_in, n_out, same, spread, double):
    """The star event, its azimuths spread and `same` outer hits moved onto the middle hit."""
    h = _star_event(n_in, n_out)
    rng = np.random.default_rng(n_out)
    phi = np.arctan2(h.y, h.x).astype(np.float64) + spread * rng.uniform(-1, 1, h.n_hits)
    r = np.hypot(h.x.astype(np.float64), h.y)
    dt = np.float64 if double else np.float32
    x, y, z = (r * np.cos(phi)).astype(dt), (r * np.sin(phi)).astype(dt), h.z.astype(dt)
    mid = n_in
    x[mid + 1:mid + 1 + same], y[mid + 1:mid + 1 + same], z[mid + 1:mid + 1 + same] = x[mid], y[mid], z[mid]
    return E.Hits(x, y, z, h.layer, h.module, h.track, h.event_offsets)


@pytest.mark.parametrize("n_in,n_out", [(9, 95), (64, 97), (65, 190), (150, 192), (150, 193), (129, 289), (70, 1030)])
@pytest.mark.parametrize("same,spread,double,theta", [(0, 1e-7, False, None), (0, 3e-3, False, None), (0, 3e-3, True, None),
                                                      (2, 3e-3, False, None), (0, 3e-3, False, 0.6)])
def test_links_at_the_edges_of_the_staged_out_cells(n_in, n_out, same, spread, double, theta):
    kw = {} if theta is None else dict(ca_theta_barrel=theta, ca_theta_endcap=theta)
    cfg_d = C.default_config(cut_mask=C.CUT_PHIW, **kw)
    h = _event(n_in, n_out, same, spread, double)
    rci, rco, _ = O.doublets(cfg_d, h.x, h.y, h.z, h.layer)
    rli, rlo = O.links(cfg_d, h.x, h.y, h.z, h.layer, rci, rco)
    ci, co, li, lo = _doublets_and_links(h, cfg_d, 1 << 17, 1 << 18)
    assert doublet_set(ci, co) == doublet_set(rci, rco)
    ref = link_set(rci, rco, rli, rlo)
    assert len(ref) > 0
    assert link_set(ci, co, li, lo) == ref
