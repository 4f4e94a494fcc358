"""The clusterizer's blocks at the sizes where they can go wrong: rows cut into several parts, parts that just fit the
digits a block holds or do not, rows of more pads than a part may have, times and charges at the ends of their types,
input arrays that allow no wide loads.  Bit for bit against the oracle (whole numbers, and FP64 expressions rounded once)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _digits(rng, half, n_units, per_pad, t_max, q_max):
    """Random digits, about per_pad(row) of them in each pad, times from the full range, many equal charges."""
    times, off = [], [0]
    for _ in range(n_units):
        for r, h in enumerate(half):
            for _ in range(2 * h):
                n = int(rng.integers(0, 2 * per_pad(r) + 1))
                t = np.unique(rng.integers(0, t_max + 1, n))
                if n > 3:
                    t = np.unique(np.concatenate([t, [0, t_max]]))
                times.append(t)
                off.append(off[-1] + len(t))
    time = np.concatenate(times).astype(np.uint16)
    q = rng.integers(8, 16, len(time)).astype(np.uint16)
    q[rng.random(len(q)) < 0.01] = q_max
    return np.asarray(off, np.int64), time, q


CASES = {  # half pads of the rows, units, digits of a pad by row, last time, largest charge
    "sparse": ([3, 4, 2], 5, lambda r: 2, 40, 1023),
    "one_part": ([8, 9], 3, lambda r: 100, 300, 1023),
    "around_the_stage": ([8, 9, 10, 11], 2, lambda r: 250 + 20 * r, 65535, 65535),
    "parts": ([8, 30, 73], 2, lambda r: 400, 4000, 1023),
    "pads_past_the_stage": ([2, 3], 2, lambda r: 4000, 9000, 1023),
    "one_long_row": ([2, 2, 2, 2, 2, 2, 150], 2, lambda r: 5, 30, 1023),
    "empty_rows": ([5, 5, 5], 3, lambda r: 300 if r == 1 else 0, 900, 1023),
}


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "odd"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_runs(name, shift):
    import torch
    import oracle
    import test_gpu_clusterizer as G
    from paper_2106_03636_amd.runtime import Clusterizer
    half, n_units, per_pad, t_max, q_max = CASES[name]
    half = np.asarray(half, np.int32)
    off, time, q = _digits(np.random.default_rng(len(name)), half, n_units, per_pad, t_max, q_max)
    print("case", name, len(time), "digits", flush=True)
    c = Clusterizer(half, G.PW, G.TB, G.ZOFF, n_units, max(1, len(time)), q_min=G.Q_MIN)
    t, qq = (torch.as_tensor(np.concatenate([np.zeros(shift, np.uint16), v]).view(np.int16)).cuda()[shift:] for v in (time, q))
    c.launch(t, qq, torch.as_tensor(off).cuda(), n_units)
    o = oracle.clusterize(half, off, time, q, n_units, G.Q_MIN, G.PW, G.TB, G.ZOFF)
    G._compare(G._host(c.result()), o, half, n_units)
