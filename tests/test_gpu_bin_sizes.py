"""The bin sort at the edges of its paths: rows a wave, a block and the
workspace sort, counts around a wave's and a block's registers, rows of one
hit and bins that hold far more hits than the rest.  Parity with the oracle,
whose tracklets change with the order of the hits inside a bin."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _compare, _Ev, T  # noqa: F401

pytestmark = pytest.mark.gpu


# alone: the event has only the three crowded rows, so their average is
# per_row and rows of more than 512 hits get a block each; otherwise the 149
# empty rows keep it below and four rows share a block
@pytest.mark.parametrize("alone, per_row, clump", [
    (False, 1, 0), (False, 64, 0), (False, 65, 0), (False, 512, 0), (False, 513, 0), (False, 2048, 0), (False, 2060, 0),
    (False, 5000, 0), (False, 300, 150), (False, 900, 150),
    (True, 513, 0), (True, 6144, 0), (True, 6150, 0), (True, 9000, 0), (True, 700, 150)])
def test_bin_sort_parity(T, alone, per_row, clump):  # noqa: F811
    import oracle
    from paper_2106_03636_amd.params import DEFAULT_PARAMS as P
    rng = np.random.default_rng(per_row + clump)
    x = synth.ROW_X_F32[10:13] if alone else synth.ROW_X_F32
    rows = np.repeat(np.arange(3) + (0 if alone else 10), per_row)
    half = x[rows].astype(np.float64) * np.tan(np.radians(10.0)) * 0.95
    y = rng.uniform(-1, 1, len(rows)) * half
    z = rng.uniform(0.0, max(20.0, per_row / 32), len(rows))
    near = np.arange(len(rows)) % per_row < clump  # these share a bin
    y[near] = rng.uniform(1.0, 1.2, near.sum())
    z[near] = rng.uniform(10.0, 10.1, near.sum())
    order = rng.permutation(len(rows))
    ev = _Ev(y[order], z[order], rows[order], [0, len(rows)], x, 0.5, "rows of %d, %d in a bin" % (per_row, clump))
    print("case bin sort", alone, per_row, clump, flush=True)
    _compare(T, ev, oracle.run_event(ev, P, fragile_eps=0.05))
