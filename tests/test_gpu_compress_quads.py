"""tpc_compress over clusters taken four at a time and one by one: arrays that
allow whole-quad accesses and arrays shifted by one element, whose every
stage is then by element; lengths around the quad, the block and the grid;
a step that is a power of two (quotient taken as a product) and one that is
not.  Against the oracle on the same tracks, compared as in
test_gpu_compress: classes and codes identical but where the oracle flags an
unrounded code within 1e-6 of a half step."""
import numpy as np
import pytest

import oracle
import synth
from conftest import cached_event, cached_oracle
from gpu_inputs import DeviceTracks

pytestmark = pytest.mark.gpu

F32 = lambda v: float(np.float32(v))  # noqa: E731


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1026, None])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("step", [1.0 / 64, 0.013])
def test_quads_and_singles(n, shift, step):
    import torch

    from paper_2106_03636_amd import make_compress_params
    from paper_2106_03636_amd.runtime import Batch, Compressor
    ev, o = cached_event("pp_sector"), cached_oracle("pp_sector")
    n = ev.n if n is None else n
    tl = o["track_tracklet"]
    ct = np.ascontiguousarray(o["cluster_track"][:n])
    par, xref = o["trk_params"][tl].astype(np.float32), o["trk_xref"][tl].astype(np.float32)
    dt = DeviceTracks(n, params=par, x_ref=xref, n_hits=np.zeros(len(tl), np.int32), cluster_track=ct)
    b = Batch(ev.y[:n], ev.z[:n], ev.row[:n], [0, n], ev.row_x, ev.bz)
    cmp = Compressor(dt, make_compress_params(step=step))

    def moved(t):  # the same values, one element further on
        m = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        m[1:].copy_(t)
        return m[1:]

    if shift:
        b.y, b.z, b.row, dt.cluster_track = moved(b.y), moved(b.z), moved(b.row), moved(dt.cluster_track)
        dt.struct.cluster_track = dt.cluster_track.data_ptr()
        cmp.o_cls, cmp.o_code_y, cmp.o_code_z = moved(cmp.o_cls), moved(cmp.o_code_y), moved(cmp.o_code_z)
    print("case quads", n, shift, step, flush=True)
    cmp.launch(b)
    g = {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in cmp.result().items()}
    cp = cmp.params
    k = F32(np.float32(-np.float32(synth.KAPPA) * np.float32(ev.bz)))
    w = oracle.compress(ev.y[:n], ev.z[:n], ev.row[:n], ct, par, xref, ev.row_x, k, F32(cp.step), F32(cp.pt_remove),
                        F32(cp.sinphi_max))
    assert np.array_equal(g["cls"], w["cls"])
    differ = (g["code_y"] != w["code_y"]) | (g["code_z"] != w["code_z"])
    assert not (differ & ~w["fragile"].astype(bool)).any()
    h, a = cp.hist_half, g["cls"] == 1
    for f, hist in (("code_y", g["hist_y"]), ("code_z", g["hist_z"])):
        c = g[f][a]
        assert np.array_equal(hist, np.bincount(c[(c >= -h) & (c < h)] + h, minlength=2 * h))
    assert g["counts"][:4].tolist() == np.bincount(g["cls"], minlength=4).tolist()
