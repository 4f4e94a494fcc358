"""The filter's short square root, reciprocal and quotient give the bits of the correctly rounded forms: the root and
the reciprocal on every float of the range that is_mid lets through (1e-25 to 1e25, the reciprocal of both signs), the
quotient on 2^32 pairs (2^-40 to 2^24 each) with either kind of reciprocal: that of the divisor, and the one refined
from the approximation its square root started with."""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SQRT, RCP, DIV_RCP, DIV_RSQ = range(4)
LO, HI = (int(np.float32(v).view(np.uint32)) for v in (1e-25, 1e25))
SIGN = 1 << 31


@pytest.fixture(scope="module")
def roots():
    from paper_2106_03636_amd import build
    if not os.path.exists(build.ROOTS_LIB):
        build.build_roots()
    fn = ctypes.CDLL(build.ROOTS_LIB).kalman_roots
    fn.argtypes, fn.restype = [ctypes.c_int, ctypes.c_ulonglong, ctypes.c_ulonglong], ctypes.c_longlong
    return fn


@pytest.mark.parametrize("what, first, count", [(SQRT, LO, HI - LO + 1), (RCP, LO, HI - LO + 1),
                                                (RCP, SIGN + LO, HI - LO + 1), (DIV_RCP, 0, 1 << 32),
                                                (DIV_RSQ, 0, 1 << 32)])
def test_bits_of_the_short_forms(roots, what, first, count):
    print("case roots", what, first, count, flush=True)
    assert roots(what, first, count) == 0
