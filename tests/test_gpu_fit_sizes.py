"""The tracklet fit on both sides of every line of its rule for the lanes a seed gets: parity with the CPU oracle."""
import pytest

pytestmark = pytest.mark.gpu


# clusters (thousands) of the lines: 32, 450, 1200, 1800 and 3000 (times 1024); about 150 clusters per primary
@pytest.mark.parametrize("primaries", [1, 120, 190, 300, 2600, 3400, 7300, 8600, 11000, 13000, 18500, 22000])
def test_fit_parity_across_sizes(primaries):
    import oracle
    import parity
    import synth
    from paper_2106_03636_amd.params import DEFAULT_PARAMS
    from paper_2106_03636_amd.runtime import Batch, Tracker
    ev = synth.event_pbpb_central(7000 + primaries, n_primaries=primaries)
    b = Batch.from_event(ev)
    tr = Tracker(b.n, b.n_units, b.n_rows)
    tr.launch(b)
    res = tr.result()
    g = parity.gpu_state(tr, res)
    o = oracle.run_event(ev, DEFAULT_PARAMS, fragile_eps=0.05)
    rep = parity.compare(g, o)
    print("primaries %d: %d clusters, %d seeds" % (primaries, ev.n, res["n_seeds"]), flush=True)
    assert rep.ok, rep.get("failures")
