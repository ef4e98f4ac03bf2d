"""Short-range evaluations that return no potential and no energy sum the
forces alone.  Leaving a sum out changes no operation of the others, so the
forces are bit for bit those of an evaluation that returns everything, for
every smoothing degree, free-space and periodic, and so are energy gradients
without dE/dq against those with it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def M():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1402_7216_amd import msm
    msm.lib()
    return msm


@pytest.mark.parametrize("split_m", range(1, 8))
@pytest.mark.parametrize("periodic", [False, True])
def test_forces_alone_are_the_forces_of_a_full_evaluation(M, split_m, periodic):
    rng = np.random.default_rng(100 + split_m)
    n, box = 777, 24.0
    x, y, z = (torch.from_numpy(rng.uniform(0, box, n).astype(np.float32)).cuda() for _ in range(3))
    q = rng.uniform(-1, 1, n)
    q = torch.from_numpy((q - q.mean()).astype(np.float32)).cuda()
    order = 4 if split_m % 2 else 6
    plan = M.Plan(n, cutoff=8.0, spacing=2.0, order=order, split_m=split_m, box_lo=(0, 0, 0), box_len=(box,) * 3,
                  periodic=periodic)
    full = plan.compute(x, y, z, q)["f"].clone()
    f = torch.full((3, n), float("nan"), device="cuda")
    rows = [M._ptr(f[d]) for d in range(3)]
    head = (plan._h, M._ptr(plan.ws), plan.ws.numel(), M._stream(), M._ptr(x), M._ptr(y), M._ptr(z), M._ptr(q))
    assert M.lib().msm_compute(*head, *rows, None, None, None) == 0
    torch.cuda.synchronize()
    assert torch.equal(f, full)

    scale = torch.full((1,), 1.5, dtype=torch.float64, device="cuda")
    dq = torch.empty(n, device="cuda")
    grads = []
    for last in (M._ptr(dq), None):
        g = torch.full((3, n), float("nan"), device="cuda")
        assert M.lib().msm_backward(*head, M._ptr(scale), *(M._ptr(g[d]) for d in range(3)), last) == 0
        grads.append(g)
    torch.cuda.synchronize()
    assert torch.isfinite(grads[0]).all() and torch.equal(grads[0], grads[1])


@pytest.mark.parametrize("n,box,periodic", [(1, 20.0, False), (900, 10.0, False), (300, 40.0, False),
                                            (2000, 28.0, False), (2000, 28.0, True), (9000, 45.0, False),
                                            (20000, 60.0, False)])
def test_small_systems_sum_their_rows_in_parts(M, n, box, periodic):
    """Blocks of 16 waves for systems of few work items: rows longer than a
    wave stages at a time (a dense box), nearly empty rows, wrapped rows, and
    one system past the limit.  Against the float64 pair sum: a term carries a
    few roundings of its own (8 x 2^-24) and the sum over k of them at most
    k 2^-24 of the sum of their sizes; roundings of random sign stay below
    2 sqrt(k) 2^-24."""
    rng = np.random.default_rng(n + periodic)
    rc = 8.0
    pos = rng.uniform(0, box, (3, n)).astype(np.float32)
    q = rng.uniform(-1, 1, n).astype(np.float32)
    plan = M.PairPlan(n, kind="shifted_force", cutoff=rc, box_lo=(0, 0, 0), box_len=(box,) * 3, periodic=periodic)
    d = plan.describe()
    assert d["short_parts"] == (4 if n <= 9000 else 1)
    out = plan.compute(*(torch.from_numpy(np.ascontiguousarray(p)).cuda() for p in pos), torch.from_numpy(q).cuda())
    p, qd = torch.from_numpy(pos).double(), torch.from_numpy(q).double()
    f, bound, phi, phib = torch.zeros(3, n).double(), torch.zeros(3, n).double(), torch.zeros(n).double(), torch.zeros(n).double()
    for i in range(0, n, 500):
        dr = p[:, i:i + 500, None] - p[:, None, :]
        if periodic:
            dr = dr - box * torch.round(dr / box)
        r = dr.pow(2).sum(0).sqrt()
        r[r >= rc] = float("inf")
        r[torch.arange(r.shape[0]), torch.arange(i, i + r.shape[0])] = float("inf")
        near = torch.isfinite(r)
        k = near.sum(1)
        fr, fs = (1 / r ** 2 - 1 / rc ** 2) / r, (1 / r ** 2 + 1 / rc ** 2) / r
        e = torch.where(near, 1 / r + torch.where(near, r, 0.) / rc ** 2 - 2 / rc, 0.)
        es = torch.where(near, 1 / r + torch.where(near, r, 0.) / rc ** 2 + 2 / rc, 0.)
        w = (8 + 2 * k.double().sqrt()) * 2.0 ** -24
        qq = qd[i:i + 500, None] * qd[None, :]
        f[:, i:i + 500] = (qq * fr * dr).sum(2)
        bound[:, i:i + 500] = (qq.abs() * fs * dr.abs()).sum(2) * w
        phi[i:i + 500] = e @ qd
        phib[i:i + 500] = (es @ qd.abs()) * w
    # the self term of the method, from a single atom of unit charge
    alone = M.PairPlan(1, kind="shifted_force", cutoff=rc, box_lo=(0, 0, 0), box_len=(box,) * 3, periodic=periodic)
    one = alone.compute(*(torch.full((1,), 1.0, device="cuda") for _ in range(4)))
    phi = phi + qd * float(one["phi"].item())
    phib = phib + phi.abs() * 2.0 ** -22 + qd.abs() * abs(float(one["phi"].item())) * 2.0 ** -22
    err = (out["f"].cpu().double() - f).abs()
    print(f"n {n} box {box}: forces {float((err / bound.clamp_min(1e-30)).max()):.2f} of the bound", flush=True)
    assert (err <= bound + f.abs() * 2.0 ** -23).all()
    assert ((out["phi"].cpu().double() - phi).abs() <= phib).all()


@pytest.mark.parametrize("copies", [1, 60])
def test_a_batch_sums_split_rows_as_each_system_alone(M, copies):
    """Three small systems as one launch of 16-wave blocks, and many copies of
    them in 4-wave blocks that take the parts in turn: the same bits."""
    from paper_1402_7216_amd import inputs
    base = [inputs.uniform_charges(n, side, seed=n, cutoff=8.0, spacing=2.5, order=4, levels=2)
            for n, side in ((700, 9.0), (1000, 20.0), (2500, 30.0))]
    systems = base * copies
    b = M.batch_for(systems)
    out = b.compute(*M.batch_to_device(systems))
    d = b.describe()
    for s in (0, 1, 2, len(systems) - 1):
        plan = M.plan_for(systems[s])
        plan.tune(d["lattice_b"], d["item_chunks_all"][s])
        assert plan.describe()["short_parts"] == 4
        o = plan.compute(*M.to_device(systems[s]))
        lo, hi = b.offsets[s], b.offsets[s + 1]
        assert torch.equal(o["f"], out["f"][:, lo:hi]) and torch.equal(o["phi"], out["phi"][lo:hi]), s
