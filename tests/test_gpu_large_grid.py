"""Charges q^0 of level-0 grids of more than 2^22 nodes (where the node index
exceeds what float reciprocals divide exactly), free space and periodic, against
a float64 anterpolation of the same atoms: atoms along every face of the box,
where a wrong index lands on the opposite face.

Tolerance: a basis value takes about ten float32 operations on values up to 6,
a weight is a product of three, and contributions are rounded to 2^-36: 1e-5
for each atom (|q| <= 1) that touches the node."""
import numpy as np
import pytest

import oracle
from paper_1402_7216_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _expected(s, lo, n, period):
    """q^0 in float64 and the number of atoms at each node (n and lo: x, y, z; grids are indexed z, y, x)."""
    q, cnt = np.zeros(n[::-1]), np.zeros(n[::-1])
    h = s.spacing
    half = s.order // 2
    for x, y, z, c in zip(s.x.astype(np.float64), s.y.astype(np.float64), s.z.astype(np.float64),
                          s.q.astype(np.float64)):
        idx, w = [], []
        for d, v in enumerate((x, y, z)):
            t = v / h
            k = np.arange(int(np.floor(t)) - half + 1, int(np.floor(t)) + half + 1)
            wd = np.array([oracle.Phi(s.order, t - i) for i in k])
            if period is not None:        # every image of a node within the stored ones
                k = np.concatenate([k + j * period[d] for j in (-1, 0, 1)])
                wd = np.tile(wd, 3)
            keep = (k >= lo[d]) & (k < lo[d] + n[d])
            idx.append(k[keep] - lo[d])
            w.append(wd[keep])
        at = np.ix_(idx[2], idx[1], idx[0])
        q[at] += c * w[2][:, None, None] * w[1][None, :, None] * w[0][None, None, :]
        cnt[at] += 1
    return q, cnt


@pytest.mark.parametrize("nodes,periodic,order", [((200, 170, 140), False, 4), ((160, 160, 160), True, 4),
                                                  ((192, 160, 176), True, 6)])
def test_charges_of_large_grids(nodes, periodic, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1402_7216_amd import msm
    print(f"case nodes {nodes} periodic {periodic} order {order}", flush=True)
    h, levels = 2.0, 5
    length = tuple(h * v for v in nodes)
    rng = np.random.default_rng(31)
    pos = rng.uniform(0.0, 1.0, size=(3, 240)) * np.asarray(length)[:, None]
    for d in range(3):                    # a third of the atoms within two nodes of each low and high face
        pos[d, 40 * 2 * d:40 * (2 * d + 1)] = rng.uniform(0.01, 4.0, 40)
        pos[d, 40 * (2 * d + 1):40 * (2 * d + 2)] = length[d] - rng.uniform(0.01, 4.0, 40)
    s = inputs._as_f32_system(pos, rng.uniform(-1.0, 1.0, 240), (0.0, 0.0, 0.0), length, cutoff=12.0, spacing=h,
                              order=order, levels=levels, name="large")
    plan = msm.plan_for(s, periodic=periodic)
    _, lo, n = plan.info()
    assert int(np.prod(n[0])) > 1 << 22
    plan.compute(*msm.to_device(s))
    torch.cuda.synchronize()
    plan.check()
    shape = tuple(int(v) for v in n[0])
    got = plan.section(msm.SECTION_QGRID)[:int(np.prod(shape))].double().cpu().numpy().reshape(shape[::-1])
    ref, cnt = _expected(s, [int(v) for v in lo[0]], shape, nodes if periodic else None)
    err = np.abs(got - ref)
    print(f"  {shape}: worst {err.max():.2e}, nodes with charge {int((cnt > 0).sum())}", flush=True)
    assert (err <= 1e-5 * cnt).all()
    assert np.abs(ref).max() > 0.1
