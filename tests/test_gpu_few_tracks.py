"""Vertices of numbers of tracks at the line between counting them per event
directly and per block of tracks (8192 tracks and 128 more for each event)."""
import pytest

pytest.importorskip("torch")

from tests import test_gpu_track_spans as spans

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("n_events,grouped", [(1, True), (300, True), (300, False)])
def test_vertices_at_the_line_between_the_counts(over, n_events, grouped):
    spans.test_vertices_of_tracks_in_any_order(8192 + 128 * n_events + over, n_events, n_events, grouped)
