"""The Fishbone where a doublet has no length, or next to none: its inner hit lies
on the outer one.  Such a doublet is aligned with every other of that outer
hit (a zero cross product), whatever their directions; hits with numbers of
doublets for each of the kernels that test them, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from synth import config as C
from synth import events as E
from tests.helpers import doublet_set

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dz", [(np.float32, 0.0), (np.float64, 0.0), (np.float64, 1e-20)])
@pytest.mark.parametrize("theta", [0.01, 0.3])
def test_fishbone_with_doublets_of_no_length(dtype, dz, theta):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests.gpu_helpers import run_chain
    rng = np.random.default_rng(5)
    counts = [2, 64, 257, 513, 1025, 3600]
    xs, ys, zs, ls = [], [], [], []
    for i, n_in in enumerate(counts):
        phi_o = -2.8 + 0.9 * i
        xo, yo = 6.8 * np.cos(phi_o), 6.8 * np.sin(phi_o)
        phi = phi_o + rng.uniform(-0.005, 0.005, n_in)
        x, y, z = 2.9 * np.cos(phi), 2.9 * np.sin(phi), rng.uniform(-4, 4, n_in)
        x[n_in // 2], y[n_in // 2], z[n_in // 2] = xo, yo, dz
        xs += [[xo], x]; ys += [[yo], y]; zs += [[0.0], z]; ls += [[1], np.zeros(n_in)]
    x, y, z = (np.concatenate(a).astype(dtype) for a in (xs, ys, zs))
    h = E.Hits(x, y, z, np.concatenate(ls).astype(np.uint8), np.zeros(len(x), np.int16), np.full(len(x), -1, np.int32),
               np.array([0, len(x)], np.int32))
    cfg = C.default_config(fishbone_theta=theta, cut_mask=C.CUT_PHIW)
    ri, ro, _ = O.doublets(cfg, h.x, h.y, h.z, h.layer)
    per_hit = np.bincount(ro, minlength=len(x))
    assert sorted(per_hit[per_hit > 0].tolist()) == counts
    keep = O.fishbone(cfg, h.x, h.y, h.z, ri, ro)
    if dz == 0.0:
        assert keep.sum() == len(counts)      # the doublets of no length alone
    pipe, _ = run_chain(h, cfg)
    ci, co, _ = (t.cpu().numpy() for t in pipe.cells.valid())
    assert doublet_set(ci, co) == doublet_set(ri[keep], ro[keep])
