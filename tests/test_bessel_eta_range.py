"""Debye's seeds use a polynomial fitted for y' = (nu - x) / (nu + x) <= kEtaYMax, nu = l + 1/2.  The
kernels take seeds for x >= 64 at l and l + 1, l = max(ltop(x), R), R the top row of the 16-row
block that holds min(ltop(x), l_max): at most ltop(x) + 16, ltop(x) = floor(x + 14.2 x^(1/3) + 9.5)."""
import ctypes
import os

import numpy as np

from test_bessel_seed_host import LIB, ltop


def test_seeds_stay_in_the_fitted_range():
    if not os.path.exists(LIB):
        from paper_2509_25110_amd import build
        build.build_hostcheck(verbose=False)
    lib = ctypes.CDLL(LIB)
    lib.los_hostcheck_eta_y_max.restype = ctypes.c_double
    bound = lib.los_hostcheck_eta_y_max()
    assert 0.4 < bound < 1.0
    for x in np.concatenate([np.arange(64.0, 400.0, 0.125), np.geomspace(400.0, 2e4, 2000)]):
        nu = ltop(x) + 16 + 0.5
        assert (nu - x) / (nu + x) <= bound, x
