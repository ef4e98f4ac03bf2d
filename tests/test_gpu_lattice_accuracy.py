"""Accuracy of the GPU lattice cutoff: u^{k,cut} of every level below the top
against a float64 convolution of the device's own q^k.

Charges of very different size (one of 1e5 among charges of 1e-3, charges of
1e-6): the error of a node is bounded by its own terms, whatever else lies near
it.  Per node, of the convolution of |q| with |W|: the sum of the rows +-ny is
rounded (2^-24), weights are held to 2^-25, three small products are dropped
(2^-24), an accumulator takes at most 6 matrix products of 32 terms before it is
flushed to float64 (6 x 4 partial sums, 2^-23 each if they are cut off), and the
result is rounded (2^-24): below 4e-6.

Water: the root mean square error is no larger than that of the same sum in
chains of float32 FMAs (one chain per row, over the x taps, of the sum of the
rows +-ny; float64 totals every four rows)."""
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


def _levels(M, s, planes, periodic=False):
    """(q, u, weights, inner) of every level below the top, evaluated on the device."""
    plan = M.plan_for(s, periodic=periodic)
    plan.tune(lattice_b=planes)
    d = plan.describe()
    assert d["lattice_b"] == planes, d
    plan.compute(*M.to_device(s))
    torch.cuda.synchronize()
    plan.check()
    levels, _, n = plan.info()
    qg = plan.section(M.SECTION_QGRID).double().cpu().numpy()
    ug = plan.section(M.SECTION_UCUT).double().cpu().numpy()
    r = np.arange(-d["halo"], d["halo"] + 1)
    dist = s.spacing * np.sqrt(r[:, None, None] ** 2 + r[None, :, None] ** 2 + r[None, None, :] ** 2)
    g0 = np.vectorize(lambda v: oracle.split_kernel(0, v, **s.params()))
    w = np.where(dist < 2.0 * s.cutoff, g0(dist), 0.0)
    off = 0
    for k in range(levels - 1):
        cnt, shape = int(np.prod(n[k])), tuple(int(v) for v in reversed(n[k]))
        yield (qg[off:off + cnt].reshape(shape), ug[off:off + cnt].reshape(shape), w * 2.0 ** -k,
               tuple(slice(d["ghost"], v - d["ghost"]) for v in shape))
        off += cnt


def _conv(q, w):
    t = torch.nn.functional.conv3d(torch.from_numpy(q)[None, None], torch.from_numpy(w)[None, None],
                                   padding=w.shape[0] // 2)
    return t[0, 0].numpy()


def _float32_chains(q, w):
    """The convolution in float32 FMAs (products of float32 are exact in float64)."""
    H = w.shape[0] // 2
    pad = np.pad(q.astype(np.float32), H)
    w = w.astype(np.float32).astype(np.float64)
    nz, ny, nx = q.shape
    total, acc, rows = np.zeros(q.shape), np.zeros(q.shape, np.float32), 0
    for dz in range(2 * H + 1):
        for ay in range(H + 1):
            if not w[dz, H + ay].any():
                continue
            both = pad[dz:dz + nz, H + ay:H + ay + ny]
            if ay:
                both = both + pad[dz:dz + nz, H - ay:H - ay + ny]
            for dx in range(2 * H + 1):
                if w[dz, H + ay, dx]:
                    acc = (acc + w[dz, H + ay, dx] * both[:, :, dx:dx + nx].astype(np.float64)).astype(np.float32)
            rows += 1
            if rows % 4 == 0:
                total += acc
                acc = np.zeros(q.shape, np.float32)
    return (total + acc).astype(np.float32)


def _charges(name):
    h, half_width = 2.0, 9
    rng = np.random.default_rng(77)
    length = np.array([40.0, 14.0, 12.0]) * h
    pos = rng.uniform(0.0, 1.0, size=(3, 400)) * length[:, None]
    q = rng.uniform(-1.0, 1.0, 400)
    if name == "one_large":
        q *= 1e-3
        q[0], pos[:, 0] = 1e5, (0.7, 13.1, 11.4)
    else:
        q *= 1e-6
    return inputs._as_f32_system(pos, q, (0.0, 0.0, 0.0), tuple(length), cutoff=0.5 * h * (half_width + 0.5),
                                 spacing=h, order=4, levels=3, name=name)


@pytest.mark.parametrize("planes", [4, 6, 8])
@pytest.mark.parametrize("name", ["one_large", "small"])
def test_error_is_bounded_by_the_terms_of_the_node(M, name, planes):
    print(f"case {name} planes {planes}", flush=True)
    for k, (q, u, w, inner) in enumerate(_levels(M, _charges(name), planes)):
        ref, size = _conv(q, w), _conv(np.abs(q), np.abs(w))
        assert np.count_nonzero(q) > q.size // 4
        err = np.abs(u - ref)[inner]
        print(f"  level {k}: {float((err / np.maximum(size, 1e-300)).max()):.2e} of the terms", flush=True)
        assert (err <= TOL * size).all()


@pytest.mark.parametrize("planes", [4, 6, 8])
@pytest.mark.parametrize("case", ["water_h11", "water_h9_quintic", "periodic_h10"])
def test_error_is_no_larger_than_float32_chains(M, case, planes):
    print(f"case {case} planes {planes}", flush=True)
    periodic = case.startswith("periodic")
    if case == "water_h11":
        s = inputs.water_box(6000, 91, cutoff=12.0, spacing=2.0, order=4, levels=3)
    elif case == "water_h9_quintic":
        s = inputs.water_box(6000, 92, cutoff=12.0, spacing=2.5, order=6, levels=3)
    else:
        s = inputs.water_box(6000, 93, cutoff=10.0, spacing=2.0, order=6, levels=3)
        s.spacing = inputs.periodic_spacing(s.box_len[0], 2.0, 3)
    for k, (q, u, w, inner) in enumerate(_levels(M, s, planes, periodic)):
        ref = _conv(q, w)[inner]
        got = np.sqrt(np.mean((u[inner] - ref) ** 2))
        chains = np.sqrt(np.mean((_float32_chains(q, w)[inner] - ref) ** 2))
        rms = np.sqrt(np.mean(ref ** 2))
        print(f"  level {k}: {got / rms:.2e}, chains {chains / rms:.2e}", flush=True)
        assert got <= chains
