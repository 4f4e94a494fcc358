"""tpc_merge_tracks on states whose x and y lie beyond the 8192 cm up to which FP32 holds them to the pair scan's
margins: the scan's first look in FP32 must leave their windows to the exact test.  Segments of one unit continue in
the next one at candidates placed around the edge of the y window; links and candidate counts are the oracle's, which
decides in FP64 from the same FP32 inputs."""
import numpy as np
import pytest

import oracle
import synth
from gpu_inputs import DeviceRefit, DeviceTracks
from test_gpu_merge import ORACLE_MERGE, _compare, _f32, _gpu_merge

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("far", [100.0, 8100.0, 5.0e4, 2.0e6])
def test_candidates_at_the_edge_of_the_window(far):
    n, n_rows = 2000, 152
    rng = np.random.default_rng(int(far))
    alpha = np.array([synth.sector_alpha(0), synth.sector_alpha(1)], np.float32)
    side = np.ones(2, np.int32)
    d = float(alpha[1]) - float(alpha[0])
    # straight outer states, far apart in y, so that each meets its own candidate only
    x = np.full(n, far).astype(np.float32).astype(np.float64)
    y = (far / 4 + 16.0 * np.arange(n) * min(1.0, far / 1.6e5)).astype(np.float32).astype(np.float64)
    if far < 1e4:
        y = (rng.uniform(-far / 4, far / 4, n)).astype(np.float32).astype(np.float64)
    phi = rng.uniform(-0.2, 0.2, n) + 0.5 * d
    s = np.sin(phi).astype(np.float32).astype(np.float64)
    # turned into the second unit's frame, and carried on by a few cm
    xq, yq = x * np.cos(d) + y * np.sin(d), -x * np.sin(d) + y * np.cos(d)
    tan = np.tan(np.arcsin(s) - d)
    xb = (xq + rng.uniform(0.5, 3.0, n)).astype(np.float32).astype(np.float64)
    dy = ORACLE_MERGE["dy_max"] * rng.choice([-1.0, 1.0], n) * (1.0 + rng.uniform(-0.1, 0.1, n))
    yb = yq + (xb - xq) * tan + dy
    p_out, p_in = np.zeros((2 * n, 5)), np.zeros((2 * n, 5))
    p_out[:n, 0], p_out[:n, 2] = y, s
    p_in[n:, 0], p_in[n:, 2] = yb, np.sin(np.arcsin(s) - d)
    p_in[:n, 0], p_in[:n, 2] = y, s
    p_out[n:] = p_in[n:]
    cov = np.zeros((2 * n, 15))
    cov[:, [0, 2, 5, 9, 14]] = 1.0
    fr, lr = np.repeat([0, 101], n), np.repeat([100, 151], n)  # the second ones end in the last row
    unit = np.repeat([0, 1], n).astype(np.int32)
    r = _f32(dict(ok=np.ones(2 * n, np.int8), p=p_in, cov=cov, x_ref=np.r_[x, xb], chi2=np.zeros(2 * n), p_out=p_out,
                  cov_out=cov, x_out=np.r_[x, xb]))
    ev = synth.Event(np.zeros(4 * n, np.float32), np.zeros(4 * n, np.float32),
                     np.stack([fr, lr], 1).reshape(-1).astype(np.uint16), np.array([0, 4 * n], np.int64),
                     np.zeros(1, np.int16), np.full(4 * n, -1, np.int32), None, 0.0, "far")
    dt = DeviceTracks(4 * n, np.arange(0, 4 * n, 2, dtype=np.int32), np.full(2 * n, 2, np.int32),
                      np.arange(4 * n, dtype=np.int32), unit=unit)
    print("case merge far", far, flush=True)
    mg = _gpu_merge(ev, dt, DeviceRefit(dt, r), alpha, side)
    g = {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in mg.result(2 * n).items()}
    o = oracle.merge(unit, fr, lr, r, alpha.astype(np.float64), side, n_rows, 0.0, **ORACLE_MERGE)
    print("pairs", g["n_pairs"], "candidates", g["n_candidates"], o["n_candidates"], "links", g["n_links"], flush=True)
    _compare(g, o)
    assert g["n_candidates"] > n // 4
