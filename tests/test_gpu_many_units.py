"""Numbers of units around the blocks that lay out their cells, chunks and
tiles (256 units a turn): parity with the oracle on slices of one sector,
some of them empty."""
import numpy as np
import pytest

from conftest import cached_event
from test_gpu_parity import _compare, _Ev, T  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_units", [1, 2, 255, 256, 257, 513])
def test_parity_of_many_units(T, n_units):  # noqa: F811
    import oracle
    from paper_2106_03636_amd.params import DEFAULT_PARAMS as P
    ev = cached_event("pp_sector")
    rng = np.random.default_rng(n_units)
    unit = rng.integers(0, max(1, min(8, n_units)), ev.n)  # the sector's clusters dealt to a few units
    unit = np.sort(rng.permutation(n_units)[: max(1, min(8, n_units))])[unit]
    order = np.argsort(unit, kind="stable")
    off = np.concatenate([[0], np.cumsum(np.bincount(unit, minlength=n_units))])
    e = _Ev(ev.y[order], ev.z[order], ev.row[order], off, ev.row_x, ev.bz, "%d units" % n_units)
    print("case units", n_units, flush=True)
    _compare(T, e, oracle.run_event(e, P, fragile_eps=0.05))
