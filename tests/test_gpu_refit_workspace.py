"""A refit needs the workspace of its own arrays (buckets and flags, an order and a packed record per track hit and
cluster), not that of the chain fit, which tpc_refit_workspace_size also covers: a call with that much gives the same
bits as one with more, one with less is refused."""
import numpy as np
import pytest

from conftest import cached_event
from gpu_inputs import DeviceTracks, truth_tracks

pytestmark = pytest.mark.gpu


def _align(b):
    return (b + 255) // 256 * 256


@pytest.mark.parametrize("n_tracks", [1, 64, 120])
def test_refit_with_a_workspace_of_its_own_size(n_tracks):
    import torch

    import paper_2106_03636_amd as T
    from paper_2106_03636_amd.runtime import Batch, Refitter, TrackingError
    ev = cached_event("pp_sector")
    first, nh, hits, _ = truth_tracks(ev)
    first, nh = first[:n_tracks], nh[:n_tracks]
    n_tracks, hits = len(nh), hits[:first[-1] + nh[-1]]
    b, dt = Batch.from_event(ev), DeviceTracks(ev.n, first, nh, hits)
    print("case refit workspace", n_tracks, len(hits), flush=True)
    rf = Refitter(dt)
    rf.launch(b)
    want = {k: v.cpu().numpy().copy() for k, v in rf.result(n_tracks).items()}
    size = _align(1280) + _align(4 * n_tracks) + _align(8 * ev.n) + _align(8 * len(hits))
    assert size <= rf.ws_bytes
    rf.workspace = torch.empty(size, dtype=torch.uint8, device="cuda")
    rf.ws_bytes = size
    rf.launch(b)
    got = rf.result(n_tracks)
    for f in want:
        assert np.array_equal(want[f], got[f].cpu().numpy()), f
    rf.ws_bytes = size - 256
    with pytest.raises(TrackingError) as e:
        rf.launch(b)
    assert e.value.status == T.TPC_E_NOMEM
