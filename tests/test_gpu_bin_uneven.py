"""The bin sort's rows that do not fit its LDS pool: a few dense rows among many sparse ones (a wave a row, the dense
ones by the whole block) and dense rows alone (a block a row), with their counters in LDS and in memory, and with a bin
so full that one wave ranks the hits.  Parity with the oracle, whose tracklets change with the order of the hits inside
a bin."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _compare, _Ev, T  # noqa: F401

pytestmark = pytest.mark.gpu

POOL = {False: 4096, True: 12288}  # LDS words of a block: sparse batch, dense batch


# alone: only the dense rows, so the batch's mean is theirs; counters: where
# they are (in LDS up to the pool's words)
@pytest.mark.parametrize("alone, per_row, clump, counters", [
    (False, 7000, 0, "lds"), (False, 7000, 60, "lds"), (False, 7000, 400, "lds"),
    (False, 14000, 0, "memory"), (False, 14000, 400, "memory"),
    (True, 9000, 400, "lds"), (True, 20000, 0, "lds"), (True, 36000, 0, "memory"), (True, 36000, 1200, "memory")])
def test_dense_rows(T, alone, per_row, clump, counters):  # noqa: F811
    import oracle
    from paper_2106_03636_amd.params import DEFAULT_PARAMS as P
    rng = np.random.default_rng(per_row + clump)
    x = synth.ROW_X_F32[10:13] if alone else synth.ROW_X_F32
    parts = []  # (y, z, row) of each unit
    for n, rows in [(per_row, np.arange(3))] if alone else [(7, np.arange(152)), (per_row, np.arange(15, 18)), (5, np.arange(152))]:
        r = np.repeat(rows, n)
        half = x[r].astype(np.float64) * np.tan(np.radians(10.0)) * 0.95
        y = rng.uniform(-1, 1, len(r)) * half
        z = rng.uniform(0.0, max(20.0, n / 32), len(r))
        near = np.arange(len(r)) % n < (clump if n == per_row else 0)  # these share a bin
        y[near] = rng.uniform(1.0, 1.2, near.sum())
        z[near] = rng.uniform(10.0, 10.1, near.sum())
        order = rng.permutation(len(r))
        parts.append((y[order], z[order], r[order]))
    y, z, row = (np.concatenate([p[i] for p in parts]) for i in range(3))
    off = np.concatenate([[0], np.cumsum([len(p[0]) for p in parts])])
    ev = _Ev(y, z, row, off, x, 0.5, "dense rows of %d, %d in a bin" % (per_row, clump))
    print("case dense rows", alone, per_row, clump, flush=True)
    g, _ = _compare(T, ev, oracle.run_event(ev, P, fragile_eps=0.05))
    count, bins = g["seg"][:, 1], g["seg"][:, 6] * g["seg"][:, 8]  # hits; bins in y times bins in z
    dense = np.flatnonzero(count == per_row)
    assert len(dense) == 3
    assert np.all(bins[dense] + 1 + per_row > POOL[alone])
    assert np.all((bins[dense] > POOL[alone]) == (counters == "memory"))
