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
