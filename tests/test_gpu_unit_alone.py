"""The bits of a unit's tracks do not depend on what else the batch holds: the tracklet fit is one of six kernels,
chosen by the number of clusters of the whole batch, and units tracked alone or among others in batches of every one
of these sizes give the same tracks, states and hits, bit for bit."""
import numpy as np
import pytest

from conftest import cached_event

pytestmark = pytest.mark.gpu

K = 1024
# lanes per seed, seeds per wave: clusters of a batch from .. to
VARIANTS = [("16 x 1", 0, 32 * K), ("16 x 4", 32 * K, 450 * K), ("8 x 8", 450 * K, 1200 * K),
            ("4 x 16", 1200 * K, 1800 * K), ("2 x 32", 1800 * K, 3000 * K), ("one a seed", 3000 * K, 1 << 30)]


def _units(ev):
    return [(ev.y[a:b], ev.z[a:b], ev.row[a:b]) for a, b in zip(ev.unit_offsets[:-1], ev.unit_offsets[1:])]


def _track(ev, units):
    """The tracks of a batch of units, as host arrays."""
    from paper_2106_03636_amd.runtime import Batch, Tracker
    off = np.concatenate([[0], np.cumsum([len(u[0]) for u in units])]).astype(np.int64)
    b = Batch(*(np.concatenate([u[i] for u in units]) for i in range(3)), off, ev.row_x, ev.bz)
    tr = Tracker(b.n, b.n_units, b.n_rows)
    tr.launch(b)
    res = tr.result()
    return b.n, {k: v.cpu().numpy() for k, v in res.items() if hasattr(v, "cpu")}


def _of_first(g, n_units, n_clusters):
    """What a batch's outputs say about its first units."""
    m = int((g["unit"] < n_units).sum())
    assert np.all(g["unit"][:m] < n_units)  # tracks come in unit order
    last = g["first_hit"][m - 1] + g["n_hits"][m - 1]
    out = {k: g[k][:m] for k in ("unit", "n_hits", "n_fit", "first_hit", "params", "cov", "x_ref", "chi2")}
    return dict(out, hits=g["hits"][:last], cluster_track=g["cluster_track"][:n_clusters])


def test_units_alone_and_in_batches_of_every_size():
    sector, central = cached_event("pp_sector"), cached_event("pbpb_central")
    one, others = _units(sector)[0], _units(central)
    assert sector.bz == central.bz and np.array_equal(sector.row_x, central.row_x)
    n, alone = _track(sector, [one])
    assert VARIANTS[0][1] < n <= VARIANTS[0][2]
    two = [len(one[0]), len(one[0]) + len(others[0][0])]  # clusters of the first unit, of the first two
    want = {1: _of_first(alone, 1, two[0])}
    assert len(want[1]["n_hits"]) > 100
    for name, lo, hi in VARIANTS[1:]:
        units, total = [one], len(one[0])
        while total <= lo or len(units) < 2:
            units.append(others[(len(units) - 1) % len(others)])
            total += len(units[-1][0])
        n, g = _track(sector, units)
        print("case units", name, len(units), "units", n, "clusters", flush=True)
        assert lo < n <= hi
        for first in (1, 2):
            got = _of_first(g, first, two[first - 1])
            ref = want.setdefault(first, got)
            for f in ref:
                assert np.array_equal(ref[f].view(np.uint8), np.ascontiguousarray(got[f]).view(np.uint8)), (name, f)
