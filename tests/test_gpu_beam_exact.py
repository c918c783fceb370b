"""The beam-spot test at the cut itself: links whose distance equals the cut to
the last bit, or misses it by one unit in the last place, which the test by
refined reciprocals leaves to the exact divisions and square roots."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from synth import config as C
from synth import events as E
from tests.helpers import link_set
from tests.test_gpu_edge import _doublets_and_links

pytestmark = pytest.mark.gpu


def _distance(h, t):
    """|distance of the circle's centre from the origin - its radius| of a triplet, operation by operation."""
    X, Y = (np.asarray(a, np.float64)[list(t)] for a in (h.x, h.y))
    ux, uy, vx, vy = X[1] - X[0], Y[1] - Y[0], X[2] - X[0], Y[2] - Y[0]
    Dd = 2.0 * (ux * vy - uy * vx)
    U2, V2 = ux * ux + uy * uy, vx * vx + vy * vy
    cx, cy = (U2 * vy - V2 * uy) / Dd, (V2 * ux - U2 * vx) / Dd
    Cx, Cy = X[0] + cx, Y[0] + cy
    return abs(np.sqrt(Cx * Cx + Cy * Cy) - np.sqrt(cx * cx + cy * cy))


@pytest.mark.parametrize("theta", [None, 0.6])     # the windowed search, the sweep
@pytest.mark.parametrize("pick", [0.1, 0.5, 0.9])
def test_links_at_the_beam_cut(theta, pick):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.Generator(np.random.PCG64(11))
    h = E.make_event(rng, n_vertices=8, fixed_tracks=30, noise_frac=0.2)
    kw = {} if theta is None else dict(ca_theta_barrel=theta, ca_theta_endcap=theta)
    cfg = C.default_config(**kw)
    ci, co, _ = O.doublets(cfg, h.x, h.y, h.z, h.layer)
    li, lo = O.links(cfg, h.x, h.y, h.z, h.layer, ci, co)
    links = sorted(link_set(ci, co, li, lo))
    t = links[int(pick * len(links))]
    at = _distance(h, t)
    for rmax, passes in ((at, True), (np.nextafter(at, 0.0), False), (np.nextafter(at, 1.0), True)):
        cfg = C.default_config(ca_rmax_bpix1=rmax, ca_rmax_other=rmax, **kw)
        ref = link_set(ci, co, *O.links(cfg, h.x, h.y, h.z, h.layer, ci, co))
        assert (t in ref) == passes
        gci, gco, gli, glo = _doublets_and_links(h, cfg, 1 << 18, 1 << 18)
        assert link_set(gci, gco, gli, glo) == ref
