"""tpc_merge_tracks on made-up segments that reach the edges of its pair scan:
fewer segments than a wave takes, waves whose segments lie in several units,
many more pairs in a wave than it buffers, a z' cell past the size sorted in
LDS, more segments than the smallest share of the grid's waves holds; states
whose direction lies below, between and above the limits (so the first look's
test in FP32 and the exact one both decide), curvatures on both sides of its
bound, units on both sides.  Against the oracle, which decides in FP64 from
the same FP32 inputs: links, candidate counts (a pair dropped by the first
look would be missing there) and chi2 as in test_gpu_merge: identical but on
segments the oracle flags, 1e-9 relative."""
import numpy as np
import pytest

import oracle
import synth
from gpu_inputs import DeviceRefit, DeviceTracks
from test_gpu_merge import ORACLE_MERGE, _compare, _f32, _gpu_merge, _k

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, z_half, wide", [(1, 10.0, 20.0), (3, 10.0, 20.0), (70, 40.0, 20.0), (700, 30.0, 20.0),
                                             (6000, 10.0, 0.3), (2600, 30.0, 20.0), (140000, 8192.0, 4.0)])
def test_pairs_of_made_up_segments(n, z_half, wide):
    rng = np.random.default_rng(n)
    bz, n_rows = 0.5, 152
    sector = [0, 1, 2, 18]
    alpha = np.array([synth.sector_alpha(s) for s in sector], np.float32)
    side = np.array([1, 1, 1, -1], np.int32)
    unit = rng.integers(0, 4, n) if n < 1000 else np.sort(rng.integers(0, 4, n))
    fr = np.where(rng.random(n) < 0.2, 0, rng.integers(0, n_rows - 2, n))
    lr = np.minimum(fr + rng.integers(1, 60, n), n_rows - 1)

    def states():
        p = np.zeros((n, 5))
        p[:, 0] = rng.uniform(-wide, wide, n)
        p[:, 2] = np.where(rng.random(n) < 0.2, rng.uniform(-0.999, 0.999, n), rng.uniform(-0.3, 0.3, n))
        p[:, 3] = rng.uniform(-1, 1, n)
        p[:, 4] = np.where(rng.random(n) < 0.1, rng.uniform(-60, 60, n), rng.uniform(-5, 5, n))
        return p

    p_in, p_out = states(), states()
    p_in[:, 1] = rng.uniform(-z_half, z_half, n)
    p_out[:, 1] = np.clip(p_in[:, 1] + rng.uniform(-20, 20, n), -8192, 8192)
    cov = np.zeros((n, 15))
    cov[:, [0, 2, 5, 9, 14]] = rng.uniform(0.5, 2.0, (n, 5))
    r = _f32(dict(ok=(rng.random(n) < 0.95).astype(np.int8), p=p_in, cov=cov, x_ref=85.0 + fr, chi2=np.zeros(n),
                  p_out=p_out, cov_out=cov, x_out=85.0 + lr))
    ev = synth.Event(np.zeros(2 * n, np.float32), np.zeros(2 * n, np.float32),
                     np.stack([fr, lr], 1).reshape(-1).astype(np.uint16), np.array([0, 2 * n], np.int64),
                     np.zeros(1, np.int16), np.full(2 * n, -1, np.int32), None, bz, "made up")
    dt = DeviceTracks(2 * n, np.arange(0, 2 * n, 2, dtype=np.int32), np.full(n, 2, np.int32),
                      np.arange(2 * n, dtype=np.int32), unit=unit.astype(np.int32))
    print("case merge scan", n, z_half, flush=True)
    mg = _gpu_merge(ev, dt, DeviceRefit(dt, r), alpha, side)
    g = {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in mg.result(n).items()}
    o = oracle.merge(unit, fr, lr, r, alpha.astype(np.float64), side, n_rows, _k(bz), **ORACLE_MERGE)
    print("pairs", g["n_pairs"], "candidates", g["n_candidates"], o["n_candidates"], "links", g["n_links"], flush=True)
    _compare(g, o)
    if n >= 700:
        assert g["n_candidates"] > 0
    if wide < 1:  # some waves met more pairs than they buffer
        assert g["n_pairs"] > 64 * n
