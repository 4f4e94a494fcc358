"""Tracks to collisions on both sides of the line where a block sums its
candidates in LDS (1024 of them), with every track in one bin, a few bins and
more bins than a wave combines; fewer tracks than a wave and many blocks'.
Against the oracle: bins, candidates and counts identical, the candidates'
mean z' within 2^-17 cm.  The tracks' own z' is test_gpu_collisions' subject,
not compared here (an almost straight one, |q/pT| 4e-7, differs by 7e-9 cm)."""
import numpy as np
import pytest

from gpu_inputs import DeviceTracks
from test_gpu_collisions import BAR_Z, T, _host, _oracle  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, vertices", [(5, 1), (64, 3), (70000, 1), (70000, 40), (70000, 511), (70000, 1500)])
def test_bins_of_tracks(T, n, vertices):  # noqa: F811
    from paper_2106_03636_amd.runtime import CollisionAssigner
    rng = np.random.default_rng(n + vertices)
    vertex = rng.integers(0, vertices, n)
    side = np.array([1, -1], np.int32)
    unit = rng.integers(0, 2, n).astype(np.int32)
    p = np.zeros((n, 5), np.float32)
    p[:, 0] = rng.uniform(-5, 5, n)
    p[:, 2] = rng.uniform(-0.3, 0.3, n)
    p[:, 3] = rng.uniform(-0.5, 0.5, n)
    p[:, 4] = rng.uniform(-5, 5, n)
    x = rng.uniform(85, 90, n).astype(np.float32)
    # vertices 4 cm apart in the middle of a bin, the tracks' z put near them
    p[:, 1] = (vertex - vertices // 2) * 4.0 + 0.5 + rng.normal(0, 0.05, n) + p[:, 3] * x
    cp = T.make_collision_params(n_min=1, c_max=0.02)
    dt = DeviceTracks(1, params=p, x_ref=x, unit=unit, n_hits=np.zeros(n, np.int32))
    print("case collision bins", n, vertices, flush=True)
    ca = CollisionAssigner(dt, cp, cap=16384)
    ca.launch(side, 0.5)
    g = _host(ca.result())
    print("candidates", g["n_collisions"], flush=True)
    o = _oracle(cp, p, x, unit, side, 0.5)
    assert o["fragile"].sum() == 0
    assert g["n_collisions"] == o["n_collisions"]
    for f in ("side", "bin", "count", "n_form", "collision"):
        assert np.array_equal(g[f], o[f]), f
    assert np.abs(g["z"] - o["c_zdca"]).max(initial=0.0) <= BAR_Z
    if vertices == 1500:
        assert g["n_collisions"] > 1024
