"""The stream layout of a plan that nobody chose one for (no GPU needed)."""
import ctypes
import json

import pytest


def _describe(n, periodic=False, **prm):
    from paper_1402_7216_amd import msm
    p = msm.make_params(periodic=periodic, **prm)
    h = ctypes.c_void_p()
    assert msm.lib().msm_plan_create(ctypes.byref(p), n, ctypes.byref(h)) == 0
    try:
        buf = ctypes.create_string_buffer(4096)
        assert msm.lib().msm_plan_describe(h, buf, 4096) == 0
        return json.loads(buf.value.decode())
    finally:
        msm.lib().msm_plan_destroy(h)


@pytest.mark.parametrize("n,side,periodic,cutoff,spacing,layout,graph", [
    (0, 20.0, False, 8.0, 2.5, 1, 2), (1, 20.0, False, 8.0, 2.5, 1, 2), (1000, 20.0, False, 8.0, 2.5, 1, 2),
    (9000, 44.8, True, 10.0, 2.8, 2, 2), (24000, 62.1, False, 12.0, 2.0, 2, 2), (99999, 100.0, False, 12.0, 2.0, 2, 2),
    (999999, 215.44, False, 12.0, 2.5, 3, 3), (999999, 216.0, True, 12.0, 3.375, 2, 2)])
def test_layout_follows_the_size(n, side, periodic, cutoff, spacing, layout, graph):
    d = _describe(n, periodic, cutoff=cutoff, spacing=spacing, order=4, levels=4 if side > 50 else 2,
                  box_lo=(0, 0, 0), box_len=(side,) * 3)
    assert d["streams"] == 3 and (d["layout"], d["graph_layout"]) == (layout, graph)
