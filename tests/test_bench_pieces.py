"""The link-pair accounting of bench.py where a hit has more out-cells than the
link search stages at once, and where some have no direction: against a walk
over the hit's pieces, on the host."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import bench
import oracle as O
from synth import config as C
from tests.test_bench_counts import _Cells
from tests.test_gpu_link_pieces import _event

PIECE, STAGED = 96, 192


def _walk(cfg, h, ci, co):
    """Pairs that the search tests, in-cell by in-cell and piece by piece."""
    x, y, z = (np.asarray(a, np.float64) for a in (h.x, h.y, h.z))
    r = np.sqrt(x * x + y * y)
    B = min(math.floor(2.0 / (math.asin(max(cfg["ca_theta_barrel"], cfg["ca_theta_endcap"])) + 1e-4)), 128)

    def bucket(c):
        dr, dz = r[co[c]] - r[ci[c]], z[co[c]] - z[ci[c]]
        if dr < 0:
            dr, dz = -dr, -dz
        dr, dz = np.float32(dr), np.float32(dz)
        if dr + abs(dz) == 0:
            return None
        return min(max(int((dz / (dr + abs(dz)) + np.float32(1)) * np.float32(0.5 * B)), 0), B - 1)

    n = 0
    for mid in range(h.n_hits):
        outs = [bucket(c) for c in np.flatnonzero(ci == mid)]
        ins = [bucket(c) for c in np.flatnonzero(co == mid)]
        whole = len(outs) + outs.count(0) + outs.count(B - 1) <= STAGED and None not in outs
        step = max(len(outs), 1) if whole else PIECE
        for p in range(0, len(outs), step):
            piece = outs[p:p + step]
            for b in ins:
                if b is None or None in piece:
                    n += len(piece)
                else:
                    n += sum(o in ((b - 1) % B, b, (b + 1) % B) for o in piece)
    return n


@pytest.mark.parametrize("n_in,n_out,same", [(9, 95, 0), (30, 190, 0), (30, 300, 0), (30, 300, 2), (20, 100, 1)])
def test_examined_pairs_of_pieces(n_in, n_out, same):
    cfg = C.default_config(cut_mask=C.CUT_PHIW)
    h = _event(n_in, n_out, same, 3e-3, False)
    ci, co, _ = O.doublets(cfg, h.x, h.y, h.z, h.layer)
    order = np.argsort(ci, kind="stable")      # grouped by inner hit, as the library's cells are
    ci, co = ci[order], co[order]
    pairs, examined = bench.link_pair_counts(_Cells(ci, co), h, cfg)
    assert pairs > 0
    assert examined == _walk(cfg, h, ci, co)
