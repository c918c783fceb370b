"""Doublets of batches on both sides of 64 events, from where the count pass takes
its work-groups in one range per XCD instead of runs of 32: few and odd
numbers of hits, empty events, every block size."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from paper_2008_13461_amd import _abi as A
from paper_2008_13461_amd import api
from synth import config as C
from synth import events as E

pytestmark = pytest.mark.gpu


def _batch(n_events, n_hits):
    """n_hits hits of one crowded event dealt to n_events events, some of them empty."""
    rng = np.random.Generator(np.random.PCG64(n_events + n_hits))
    h = E.make_event(rng, n_vertices=1 + n_hits // 60, fixed_tracks=30, noise_frac=0.2)
    cut = np.sort(rng.integers(0, n_hits + 1, n_events - 1))
    off = np.concatenate([[0], cut, [n_hits]]).astype(np.int32)
    return E.Hits(*(getattr(h, k)[:n_hits] for k in ("x", "y", "z", "layer", "module", "track")), event_offsets=off)


@pytest.mark.parametrize("block", [64, 128, 256, 512])
@pytest.mark.parametrize("n_events", [63, 64, 65])
@pytest.mark.parametrize("n_hits", [1, 7, 257, 4001])
def test_doublets_of_many_events(n_events, n_hits, block):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = _batch(n_events, n_hits)
    cfg_d = C.default_config()
    cfg = A.make_config(cfg_d, block_doublets=block)
    cells, status = api.Cells.empty(1 << 17, n_hits), api.new_status()
    ws = api.new_workspace(api.workspace_size(cfg, n_hits, n_events, cells.cap, 16, 16))
    api.build_doublets(api.Hits.from_host(h), cfg, cells, status, ws)
    assert int(status[0].item()) == 0
    want = []
    for a, b in zip(h.event_offsets[:-1], h.event_offsets[1:]):
        i, o, p = O.doublets(cfg_d, h.x[a:b], h.y[a:b], h.z[a:b], h.layer[a:b])
        want += [(x + a, y + a, q) for x, y, q in zip(i, o, p)]
    got = list(zip(*(t.cpu().tolist() for t in cells.valid())))
    assert len(got) == len(set(got)) and set(got) == set(want)
