"""Plans that msm_compute_static takes: many atoms on a small periodic grid,
whose workspace without the lattice cutoff's partials is just below 64 MiB.
The size is checked before the (null) arrays are (no GPU needed)."""
import ctypes

import pytest

PLANS = [(8.0, 1.5, 4, 3, 48.0, 1293116), (10.0, 1.5, 4, 5, 48.0, 1229800), (13.7, 2.0, 4, 5, 32.0, 1200299),
         (13.7, 2.0, 4, 4, 48.0, 1261106), (6.5, 1.5, 4, 2, 51.0, 1340547)]


def _static(periodic, cutoff, spacing, order, levels, side, n):
    from paper_1402_7216_amd import msm
    p = msm.make_params(cutoff, spacing, order=order, levels=levels, box_len=(side,) * 3, periodic=periodic)
    h = ctypes.c_void_p()
    assert msm.lib().msm_plan_create(ctypes.byref(p), n, ctypes.byref(h)) == 0
    try:
        return msm.lib().msm_compute_static(h, None, *([None] * 10)), msm
    finally:
        msm.lib().msm_plan_destroy(h)


@pytest.mark.parametrize("plan", PLANS)
def test_dense_periodic_plans_fit_the_static_array(plan):
    code, msm = _static(True, *plan)
    assert code == msm.ERR_INVALID_ARG, msm.lib().msm_last_error()


def test_larger_plans_are_refused():
    code, msm = _static(True, 8.0, 1.5, 4, 3, 48.0, 1500000)
    assert code == msm.ERR_UNSUPPORTED
