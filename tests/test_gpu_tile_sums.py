"""The listings in a build whose work-groups never read another tile's state:
each sums the tiles before its own itself, as it does in the library when a
state is not there after a bounded number of reads.  The products equal the
library's bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2008_13461_amd import _abi as A
from paper_2008_13461_amd import api
from synth import config as C
from synth import events as E
from tests.native.build import TILES_LIB
from tests.test_gpu_tiles import _event, _run

pytestmark = pytest.mark.gpu


def _both(monkeypatch, f):
    """f() with the library and with the build that sums for itself."""
    want = f()
    monkeypatch.setattr(A, "_lib", None)   # put back after the test
    A.load(TILES_LIB)
    return want, f()


@pytest.mark.parametrize("n_hits,cells_cap,shifted", [(4097, 256 * 4097, False), (8193, 256 * 8193, True),
                                                      (8193, (1 << 24) + 1, False)])
def test_listings_without_the_states(monkeypatch, n_hits, cells_cap, shifted):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = _event(n_hits)
    want, got = _both(monkeypatch, lambda: _run(h, cells_cap, shifted))
    # tiles of 4096 doublets and of 1024 rows: more than one of each
    assert len(want[0]) > 3 * 4096 and len(want[8]) > 1024
    assert all(np.array_equal(a, b) for a, b in zip(want, got))


def test_fishbone_without_the_states(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = E.overlap_batch(n_events=2)
    hits = api.Hits.from_host(h)
    cfg = A.make_config(C.default_config(fishbone_theta=0.01))
    cap = 128 * h.n_hits

    def run():
        cells, status = api.Cells.empty(cap, h.n_hits), api.new_status()
        ws = api.new_workspace(api.workspace_size(cfg, h.n_hits, h.n_events, cap, 16, 16))
        api.build_doublets(hits, cfg, cells, status, ws)
        assert int(status[0].item()) == 0
        return [t.cpu().numpy() for t in (*cells.valid(), cells.inner_count)]

    want, got = _both(monkeypatch, run)
    assert len(want[0]) > 3 * 4096
    assert all(np.array_equal(a, b) for a, b in zip(want, got))
