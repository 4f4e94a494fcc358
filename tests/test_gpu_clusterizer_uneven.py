"""Batches whose digits lie in few of their units, rows or pads: every row is cut into the same number of parts, so the
parts of the dense ones hold more than a block stages and are taken a run of pads at a time: runs that fit, single pads
that do not, and both in one part; parts of more pads than a run may have.  Bit for bit against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pads(half, n_units, digits):
    """digits(u, r, p): mean digits of a pad, as an array over (unit, row, pad)."""
    return np.asarray([digits(u, r, p) for u in range(n_units) for r, h in enumerate(half) for p in range(2 * h)], float)


CASES = {  # half pads of the rows, units, mean digits of a pad
    "one_unit_of_many": ([30, 40, 50], 8, lambda u, r, p: 600 if u == 3 else 1),
    "last_unit": ([30, 40], 6, lambda u, r, p: 700 if u == 5 else 0),
    "one_row": ([30] * 12, 2, lambda u, r, p: 500 if r == 4 else 2),
    "hot_end_of_rows": ([40] * 6, 2, lambda u, r, p: 1500 if p > 70 else 3),
    "single_pads": ([20] * 8, 2, lambda u, r, p: 7000 if p in (0, 5, 6, 13, 39) and r % 3 == 0 else 40),
    "long_row": ([2] * 12 + [150], 2, lambda u, r, p: 400 if r == 12 and p > 100 else 2),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_uneven(name):
    import torch
    import oracle
    import test_gpu_clusterizer as G
    from paper_2106_03636_amd.runtime import Clusterizer
    half, n_units, digits = CASES[name]
    half = np.asarray(half, np.int32)
    rng = np.random.default_rng(len(name))
    times = []
    for m in rng.poisson(_pads(half, n_units, digits)):
        times.append(np.sort(rng.choice(min(65536, 3 * m + 10), m, replace=False)))
    off = np.concatenate([[0], np.cumsum([len(t) for t in times])]).astype(np.int64)
    time = np.concatenate(times).astype(np.uint16)
    q = rng.integers(8, 20, len(time)).astype(np.uint16)
    print("case", name, len(time), "digits", flush=True)
    c = Clusterizer(half, G.PW, G.TB, G.ZOFF, n_units, max(1, len(time)), q_min=G.Q_MIN)
    c.launch(*(torch.as_tensor(v.view(np.int16)).cuda() for v in (time, q)), torch.as_tensor(off).cuda(), n_units)
    o = oracle.clusterize(half, off, time, q, n_units, G.Q_MIN, G.PW, G.TB, G.ZOFF)
    G._compare(G._host(c.result()), o, half, n_units)
    # times that do not increase, wherever they lie, and a malformed offset
    import paper_2106_03636_amd as T
    from paper_2106_03636_amd.runtime import TrackingError
    dense = np.nonzero(np.diff(off) > 300)[0]
    for pad in (dense[0], dense[-1]):
        bad = time.copy()
        k = int(rng.integers(off[pad] + 1, off[pad + 1]))
        bad[k] = bad[k - 1]
        c.launch(*(torch.as_tensor(v.view(np.int16)).cuda() for v in (bad, q)), torch.as_tensor(off).cuda(), n_units)
        with pytest.raises(TrackingError) as e:
            c.result()
        assert e.value.status == T.TPC_E_INVALID
        wrong = off.copy()
        wrong[pad] = wrong[pad + 1] + 1
        c.launch(*(torch.as_tensor(v.view(np.int16)).cuda() for v in (time, q)), torch.as_tensor(wrong).cuda(), n_units)
        with pytest.raises(TrackingError) as e:
            c.result()
        assert e.value.status == T.TPC_E_INVALID
