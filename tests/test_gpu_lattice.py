"""GPU lattice cutoff (matrix-core kernel) on its own: u^{k,cut} of every level
below the top against a float64 convolution of the device's own q^k with the
stencil W(n) = 2^-k g^0(h |n|), |n| < 2a/h, at the edges of its range: stencil
half-widths 1, 8 (no wings), 9 and 13 (the widest), node counts that end
exactly on a 16-node tile, one node past it and inside the first, boxes longer
in one direction, every number of planes per block, charges far from 1, and
periodic levels.

Tolerance per node: weights and inputs are split into two float16 numbers with
at most 2^-22 of each value left over, and the product of the low parts (at
most 2^-22) is dropped: 3 2^-22; a float32 accumulator takes at most 2 rows x
(3 + 3) products x 4 planes = 48 additions before it is flushed to float64: 48
2^-24 if all err the same way; and 2^-24 for the stored result.  Together below
4e-6 of the same convolution of |q| with |W|.  A float16 number has no digits
below 2^-24, and the largest value is scaled to 2^13 or more, so a split value
also misses up to 2^-38 of the largest: over all taps, 2^-38 (max |q| sum |W| +
taps max |q| max |W|).  Typical errors are a hundred times smaller.
"""
import numpy as np
import pytest

import oracle
from paper_1402_7216_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 4e-6


@pytest.fixture(scope="module")
def M():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1402_7216_amd import msm
    msm.lib()
    return msm


def _system(half_width, box_h, seed, order=4, scale=1.0, levels=3):
    """300 random charges; spacing 2, 2a/h half-way between half_width and half_width + 1."""
    h = 2.0
    L = np.asarray(box_h, dtype=np.float64) * h
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0.0, 1.0, size=(3, 300)) * L[:, None]
    q = rng.uniform(-1.0, 1.0, size=300) * scale
    return inputs._as_f32_system(pos, q, (0.0, 0.0, 0.0), tuple(L), cutoff=0.5 * h * (half_width + 0.5), spacing=h,
                                 order=order, levels=levels, name=f"lat{half_width}")


def _conv(q, w):
    """sum_n w[n] q[mu + n] on the nodes of q, zero outside (float64)."""
    t = torch.nn.functional.conv3d(torch.from_numpy(q)[None, None], torch.from_numpy(w)[None, None],
                                   padding=w.shape[0] // 2)
    return t[0, 0].numpy()


CASES = {
    "h1": dict(half_width=1, box_h=(12, 13, 11)),
    "h8_tile_edge": dict(half_width=8, box_h=(12, 28, 12)),
    "h8_past_edge": dict(half_width=8, box_h=(13, 13, 29), order=6),
    "h9_wings": dict(half_width=9, box_h=(28, 13, 15)),
    "h13_widest": dict(half_width=13, box_h=(29, 20, 8)),
    "h9_tiny_charges": dict(half_width=9, box_h=(17, 12, 12), scale=1e-20),
    "h9_large_charges": dict(half_width=9, box_h=(17, 12, 12), scale=1e4),
    "h8_periodic": dict(half_width=8, box_h=(20, 24, 32), periodic=True),
    "h9_periodic": dict(half_width=9, box_h=(32, 20, 24), order=6, periodic=True),
    "h13_periodic": dict(half_width=13, box_h=(28, 32, 36), periodic=True),
}


@pytest.mark.parametrize("planes", [4, 6, 8])
@pytest.mark.parametrize("name", list(CASES))
def test_lattice_cutoff_matches_convolution(M, name, planes):
    c = dict(CASES[name])
    periodic = c.pop("periodic", False)
    s = _system(seed=900 + planes, **c)
    print(f"case {name} planes {planes}", flush=True)
    plan = M.plan_for(s, periodic=periodic)
    plan.tune(lattice_b=planes)
    d = plan.describe()
    assert d["lattice_b"] == planes and d["halo"] == c["half_width"], d
    plan.compute(*M.to_device(s))
    torch.cuda.synchronize()
    plan.check()
    levels, _, n = plan.info()
    qg = plan.section(M.SECTION_QGRID).double().cpu().numpy()
    ug = plan.section(M.SECTION_UCUT).double().cpu().numpy()
    H, ghost = d["halo"], d["ghost"]
    r = np.arange(-H, H + 1)
    dist = s.spacing * np.sqrt(r[:, None, None] ** 2 + r[None, :, None] ** 2 + r[None, None, :] ** 2)
    g0 = np.vectorize(lambda v: oracle.split_kernel(0, v, **s.params()))
    off = 0
    for k in range(levels - 1):
        cnt, shape = int(np.prod(n[k])), tuple(int(v) for v in reversed(n[k]))
        q, u = qg[off:off + cnt].reshape(shape), ug[off:off + cnt].reshape(shape)
        off += cnt
        w = np.where(dist < 2.0 * s.cutoff, g0(dist), 0.0) * 2.0 ** -k
        ref, size = _conv(q, w), _conv(np.abs(q), np.abs(w))
        inner = tuple(slice(ghost, v - ghost) for v in shape)
        floor = 2.0 ** -38 * np.abs(q).max() * (np.abs(w).sum() + np.count_nonzero(w) * np.abs(w).max())
        err = np.abs(u - ref)[inner]
        print(f"  level {k} {shape}: worst error {float(err.max() / size[inner].max()):.2e} of the largest sum of "
              f"magnitudes, {float((err / (TOL * size[inner] + floor)).max()):.2e} of the tolerance", flush=True)
        assert np.isfinite(u[inner]).all()
        assert (err <= TOL * size[inner] + floor).all()
