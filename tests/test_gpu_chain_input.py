"""Malformed inputs of the chain fit that its kernels meet before the status is known: each gives TPC_E_INVALID and
reads nothing outside its arrays."""
import numpy as np
import pytest

from gpu_inputs import DeviceTracks

pytestmark = pytest.mark.gpu


def _three(unit=(0, 0, 0), hits=range(6)):
    """Three segments of two hits each."""
    import test_gpu_merge as G
    seg = [0.0] * 5
    ev, _, _ = G._hand_tracks([0, 0, 0], [(0, 10), (11, 40), (50, 60)], [seg] * 3, [seg] * 3)
    return ev, DeviceTracks(ev.n, np.arange(0, 6, 2), np.full(3, 2), np.asarray(list(hits)), unit=np.asarray(unit))


@pytest.mark.parametrize("unit", [(5, 0, 0), (0, 5, 0), (0, 0, 5), (1 << 30, 0, 0), (0, 1 << 30, 0), (0, -(1 << 30), 0),
                                  (-1, 0, 0), (0, 0, -(1 << 31)), (1 << 30, -(1 << 30), 0)], ids=str)
def test_chain_segments_of_units_out_of_range(unit):
    import paper_2106_03636_amd as T
    import test_gpu_merge as G
    ev, dt = _three(unit)
    print("case chain units", unit, flush=True)
    assert G._chain_status(ev, dt, [1, 2, -1], [-1, 0, 1], [0.0]) == T.TPC_E_INVALID


@pytest.mark.parametrize("n_tracks", [0, 1, 3])
def test_hits_of_no_track_are_checked(n_tracks):
    """A hit naming no cluster is an error whether the call's tracks hold it or not, also when there are no tracks."""
    import paper_2106_03636_amd as T
    import test_gpu_merge as G
    for hits, want in ((range(6), 0), ([0, 1, 2, 3, 4, 99], T.TPC_E_INVALID), ([0, 1, 2, 3, -1, 5], T.TPC_E_INVALID)):
        ev, dt = _three(hits=hits)
        dt.counts[0] = n_tracks
        print("case chain hits", n_tracks, list(hits), flush=True)
        assert G._chain_status(ev, dt, [-1, -1, -1], [-1, -1, -1], [0.0]) == want
