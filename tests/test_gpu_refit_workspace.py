"""The refit and the chain fit work in a workspace of the refit's arrays (buckets and flags, an order, a packed record
per track hit and cluster): with exactly that much they give the bits they give with more and write nothing past it,
with less they are refused."""
import numpy as np
import pytest

from conftest import cached_event
from gpu_inputs import DeviceMerged, DeviceTracks, truth_tracks

pytestmark = pytest.mark.gpu


def _align(b):
    return (b + 255) // 256 * 256


def _host(r):
    return {k: v.cpu().numpy().copy() for k, v in r.items()}


@pytest.mark.parametrize("chains", [False, True], ids=["refit", "chains"])
@pytest.mark.parametrize("n_tracks", [2, 64, 120])
def test_a_workspace_of_the_exact_size(n_tracks, chains):
    import torch

    import paper_2106_03636_amd as T
    from paper_2106_03636_amd.runtime import Batch, ChainFitter, Refitter, TrackingError
    ev = cached_event("pp_sector")
    first, nh, hits, _ = truth_tracks(ev)
    first, nh = first[:n_tracks // 2], nh[:n_tracks // 2]
    hits = hits[:first[-1] + nh[-1]]
    nh = np.stack([nh // 2, nh - nh // 2], 1).reshape(-1)  # each track cut into two segments, which chain up
    first, n_tracks = np.cumsum(nh) - nh, len(nh)
    b = Batch.from_event(ev)
    dt = DeviceTracks(ev.n, first, nh, hits, unit=np.zeros(n_tracks))
    fit = (ChainFitter if chains else Refitter)(dt)
    at = np.arange(n_tracks)
    merged = DeviceMerged(np.where(at % 2 == 0, at + 1, -1), np.where(at % 2 == 0, -1, at - 1))
    alpha = torch.zeros(1, device="cuda")

    def launch():
        fit.launch(*((b, merged, alpha) if chains else (b,)))

    print("case workspace", n_tracks, len(hits), chains, flush=True)
    size = _align(1280) + _align(4 * n_tracks) + _align(8 * ev.n) + _align(8 * len(hits))
    assert size == fit.ws_bytes
    launch()
    want = _host(fit.result(n_tracks))
    assert want["ok"].any()
    fit.workspace = torch.full((size + 4096,), 77, dtype=torch.uint8, device="cuda")
    launch()
    got = _host(fit.result(n_tracks))
    for f in want:
        assert np.array_equal(want[f], got[f]), f
    assert bool((fit.workspace[size:] == 77).all())
    fit.ws_bytes = size - 1
    with pytest.raises(TrackingError) as e:
        launch()
    assert e.value.status == T.TPC_E_NOMEM
