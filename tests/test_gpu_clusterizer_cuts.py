"""The clusterizer's cuts of rows into parts of like many digits: more rows than one turn of the set-up's blocks, a row of
more parts than a thread writes by itself, rows of more pads than a wave holds offsets of, parts of more pads and of more
candidates than a block keeps, no room for more than a part a row, batches with no digit or with all in one pad.  Bit for
bit against the oracle; offsets out of order at the start of a row are refused."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = {  # half pads of the rows, units, mean digits of a pad
    "many_rows": ([3, 5, 4], 3000, lambda u, r, p: 6 if u % 97 == 5 else 1),
    "row_of_many_parts": ([20] * 20, 1, lambda u, r, p: 800 if r == 7 else 2),
    "long_rows": ([150, 65, 64, 63, 400], 2, lambda u, r, p: 12 if 90 < p < 300 else 1),
    "sparse_long_rows": ([150] * 30, 2, lambda u, r, p: 60 if u == 1 and r < 2 else 0.2),
    "many_candidates": ([40] * 60, 1, lambda u, r, p: 120),
    "many_candidates_and_blocks": ([40] * 76, 8, lambda u, r, p: 50),
    "two_pads_a_row": ([1] * 40, 3, lambda u, r, p: 300 if r % 5 == 0 else 20),
    "no_digits": ([30] * 5, 2, lambda u, r, p: 0),
    "one_pad": ([30] * 5, 2, lambda u, r, p: 3000 if (u, r, p) == (1, 2, 17) else 0),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_cuts(name):
    import torch
    import oracle
    import paper_2106_03636_amd as T
    import test_gpu_clusterizer as G
    from paper_2106_03636_amd.runtime import Clusterizer, TrackingError
    half, n_units, digits = CASES[name]
    half = np.asarray(half, np.int32)
    rng = np.random.default_rng(len(name))
    mean = np.asarray([digits(u, r, p) for u in range(n_units) for r, h in enumerate(half) for p in range(2 * h)], float)
    count = rng.poisson(mean)
    off = np.concatenate([[0], np.cumsum(count)]).astype(np.int64)
    gaps = rng.integers(1, 4, off[-1])
    total = np.concatenate([[0], np.cumsum(gaps)])
    pad = np.repeat(np.arange(len(count)), count)
    time = (total[1:] - total[off[pad]]).astype(np.uint16)
    q = rng.integers(8, 20, len(time)).astype(np.uint16)
    print("case", name, len(time), "digits", flush=True)
    c = Clusterizer(half, G.PW, G.TB, G.ZOFF, n_units, max(1, len(time)), q_min=G.Q_MIN)
    dev = [torch.as_tensor(v.view(np.int16)).cuda() for v in (time, q)]
    c.launch(*dev, torch.as_tensor(off).cuda(), n_units)
    o = oracle.clusterize(half, off, time, q, n_units, G.Q_MIN, G.PW, G.TB, G.ZOFF)
    G._compare(G._host(c.result()), o, half, n_units)
    # the offset at a row's start below the one before it, above the one after it, negative, past the digits; the first not 0
    start = int(2 * half[0])  # row 1 of unit 0
    for at, value in ((start, -1), (start, len(time) + 1), (start, off[start + 1] + 1), (0, 1), (start, off[start - 1] - 1)):
        wrong = off.copy()
        wrong[at] = value
        c.launch(*dev, torch.as_tensor(wrong).cuda(), n_units)
        with pytest.raises(TrackingError) as e:
            c.result()
        assert e.value.status == T.TPC_E_INVALID
