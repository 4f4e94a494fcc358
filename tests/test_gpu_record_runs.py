"""The refit and the chain fit read their hits' records eight at a time: runs whose lengths lie around multiples of
eight, at odd places of the hit list, in waves that are nearly empty or one over full; chains whose segments begin
inside and at the edge of such a group; hit lists that leave gaps, and lists that overlap (more records than the hit
list has room for).  A track's fit depends on its own hits alone, so every arrangement gives the same bits; one of
them is compared with the oracle at the fit's bars."""
import numpy as np
import pytest

import oracle
from conftest import cached_event
from gpu_inputs import DeviceTracks, truth_tracks

pytestmark = pytest.mark.gpu

LENGTHS = [3, 4, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 33, 64, 65, 100]


def _tracks(n_tracks):
    """Truth tracks of the pp sector cut to the lengths above, as lists of hits."""
    ev = cached_event("pp_sector")
    first, nh, hits, _ = truth_tracks(ev)
    out = []
    for i in range(n_tracks):
        t = i % len(nh)
        n = min(int(nh[t]), LENGTHS[i % len(LENGTHS)])
        out.append(hits[first[t]:first[t] + n])
    return ev, out


def _lists(runs, gap):
    """Hit lists one after the other with `gap` hits of nobody between them."""
    first, pos, cat = [], 0, []
    for r in runs:
        cat += [np.zeros(gap, np.int32), r]
        first.append(pos + gap)
        pos += gap + len(r)
    return np.asarray(first, np.int32), np.asarray([len(r) for r in runs], np.int32), np.concatenate(cat).astype(np.int32)


def _host(r):
    return {k: v.cpu().numpy() for k, v in r.items()}


@pytest.mark.parametrize("n_tracks", [1, 63, 64, 65, 129])
def test_refit_runs(n_tracks):
    import test_gpu_refit as R
    ev, runs = _tracks(n_tracks)
    got = []
    for gap in (0, 1, 3):
        rf, n = R._gpu_refit(ev, *_lists(runs, gap))
        got.append(_host(rf.result(n)))
    rf, n = R._gpu_refit(ev, *_lists(runs[::-1], 1))
    back = _host(rf.result(n))
    for f in got[0]:
        for other in got[1:]:
            assert np.array_equal(got[0][f], other[f]), f
        assert np.array_equal(got[0][f], back[f][::-1]), f
    R._compare(got[0], R._oracle_refit(ev, *_lists(runs, 0)), min_ok=0.75)


def _cut(run, at):
    return [r for r in np.split(run, [a for a in at if a < len(run)]) if len(r)]


@pytest.mark.parametrize("at", [(1,), (8,), (7, 16), (3, 5, 24, 25)], ids=str)
def test_chain_runs(at):
    import test_gpu_merge as G
    from parity import ParityReport, compare_fit
    ev, tracks = _tracks(70)
    tracks = [t for t in tracks if len(_cut(t, at)) > 1]
    segs, nxt, prv = [], [], []
    for t in tracks:
        parts = _cut(t, at)
        k = len(segs)
        nxt += [k + i + 1 for i in range(len(parts) - 1)] + [-1]
        prv += [-1] + [k + i for i in range(len(parts) - 1)]
        segs += parts
    alpha = np.zeros(1, np.float32)

    def fit(first, nh, hits, nx, pv):
        dt = DeviceTracks(ev.n, first, nh, hits, unit=np.zeros(len(nh)))
        return _host(G._chain_fit(ev, dt, nx, pv, alpha).result(dt.T))

    plain = fit(*_lists(segs, 0), nxt, prv)
    gaps = fit(*_lists(segs, 1), nxt, prv)
    first, nh, hits = _lists(segs, 0)
    T = len(segs)
    twice = fit(np.tile(first, 2), np.tile(nh, 2), hits, nxt + [x + T if x >= 0 else -1 for x in nxt],
                prv + [x + T if x >= 0 else -1 for x in prv])
    for f in plain:
        assert np.array_equal(plain[f], gaps[f]), f
        assert np.array_equal(plain[f], twice[f][:T]) and np.array_equal(plain[f], twice[f][T:]), f
    heads, cf, cn, ch, cu = oracle.chains(np.asarray(nxt), np.asarray(prv), first, nh, hits, np.zeros(T))
    o = oracle.refit_chains(cf, cn, ch, cu, ev.y, ev.z, ev.row, ev.row_x.astype(np.float64), np.zeros(1), G._k(ev.bz), G.P)
    gok, ook = plain["ok"][heads].astype(bool), o["ok"].astype(bool)
    assert np.array_equal(plain["n_hits"][heads], cn) and np.array_equal(gok, ook)
    both, h = gok & ook, heads[gok & ook]
    rep = ParityReport()
    compare_fit(rep, plain["params"][h], plain["cov"][h], plain["chi2"][h], plain["x_ref"][h], o["p"][both], o["cov"][both],
                o["chi2"][both], o["x_ref"][both], refit_cov0=[float(np.float32(v)) for v in G.P["cov0"]], chain=True)
    assert rep.ok, dict(rep)
