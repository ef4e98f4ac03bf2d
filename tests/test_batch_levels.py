"""Batches whose largest system has a single level (no lattice cutoff): the
others, with stencils and grids of different size, share one lattice template,
its window and its tiles.  On the CPU the launch is compared with that of the
batch without the one-level system; on the GPU the results with the oracle."""
import ctypes
import json

import numpy as np
import pytest

import oracle
from paper_1402_7216_amd import inputs
from _helpers import ENERGY_RTOL, FORCE_RTOL, PHI_RTOL, rel_rms


def _systems(order=4):
    one = inputs.uniform_charges(4000, side=24.0, seed=41, cutoff=8.0, spacing=4.0, order=order, levels=1)
    wide = inputs.uniform_charges(500, side=30.0, seed=42, cutoff=13.2, spacing=2.0, order=order, levels=2)
    grid = inputs.uniform_charges(3000, side=80.0, seed=43, cutoff=8.4, spacing=2.0, order=order, levels=4)
    return one, wide, grid


def _describe(systems):
    from paper_1402_7216_amd import msm
    prm = (msm.Params * len(systems))(*[msm.make_params(**s.params()) for s in systems])
    n = (ctypes.c_int32 * len(systems))(*[s.n for s in systems])
    h = ctypes.c_void_p()
    assert msm.lib().msm_batch_create(prm, n, len(systems), ctypes.byref(h)) == 0
    try:
        buf = ctypes.create_string_buffer(8192)
        assert msm.lib().msm_batch_describe(h, buf, 8192) == 0
        return json.loads(buf.value.decode())
    finally:
        msm.lib().msm_batch_destroy(h)


@pytest.mark.parametrize("at", [0, 1, 2])
def test_one_level_systems_leave_the_lattice_launch_alone(at):
    one, wide, grid = _systems()
    systems = [wide, grid]
    ref = _describe(systems)
    systems.insert(at, one)
    d = _describe(systems)
    assert d["lattice_b"] == ref["lattice_b"] and d["lattice_lds"] == ref["lattice_lds"]
    assert d["blocks"]["lattice"] == ref["blocks"]["lattice"]


def test_batch_of_one_level_systems_has_no_lattice_launch():
    one = _systems()[0]
    d = _describe([one, one])
    assert d["lattice_b"] == 0 and d["blocks"]["lattice"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("order", [4, 6])
def test_batch_with_a_large_one_level_system_matches_oracle(order):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1402_7216_amd import msm
    systems = list(_systems(order))
    print(f"case one-level batch order {order}", flush=True)
    b = msm.batch_for(systems)
    out = b.compute(*msm.batch_to_device(systems))
    torch.cuda.synchronize()
    b.check()
    for s, sys_ in enumerate(systems):
        a, e = b.offsets[s], b.offsets[s + 1]
        r = oracle.system_msm(sys_)
        # (random charges: the energy is a small difference of its terms)
        de = abs(out["energy"][s].item() - r["energy"]) / (0.5 * np.abs(sys_.q.astype(np.float64) * r["phi"]).sum())
        df = rel_rms(out["f"][:, a:e].double().cpu().numpy(), r["f"])
        dp = rel_rms(out["phi"][a:e].double().cpu().numpy(), r["phi"])
        print(f"  system {s}: energy {de:.2e} forces {df:.2e} phi {dp:.2e}", flush=True)
        assert de <= ENERGY_RTOL and df <= FORCE_RTOL and dp <= PHI_RTOL, s
