"""Two threads, each on a stream and a workspace of its own, evaluate one plan
(one batch) at the same time: every result equals that of a call alone.  The
systems are those whose short range is enqueued on the side stream after the
restriction, with its fork recorded before."""
import ctypes
import threading

import pytest

from paper_1402_7216_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def M():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1402_7216_amd import msm
    msm.lib()
    return msm


def _run(M, owner, compute, workspace_init, arrays, n, n_energy, rounds):
    """rounds evaluations of each of two inputs, in two threads; their results."""
    dev = owner.ws.device

    def outputs():
        return (torch.full((3, n), float("nan"), device=dev), torch.full((n,), float("nan"), device=dev),
                torch.full((n_energy,), float("nan"), dtype=torch.float64, device=dev))

    def evaluate(ws, stream, a, o):
        f, phi, e = o
        M._check(compute(owner._h, M._ptr(ws), ws.numel(), ctypes.c_void_p(stream.cuda_stream), *map(M._ptr, a),
                         M._ptr(f[0]), M._ptr(f[1]), M._ptr(f[2]), M._ptr(phi), M._ptr(e), None))

    results, errors = [[], []], []
    workspaces = [owner.ws, torch.empty_like(owner.ws)]
    M._check(workspace_init(owner._h, M._ptr(workspaces[1]), workspaces[1].numel(), M._stream()))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[outputs() for _ in range(rounds)] for _ in range(2)]
    torch.cuda.synchronize()

    def work(t):
        try:
            for o in outs[t]:
                evaluate(workspaces[t], streams[t], arrays[t], o)
            streams[t].synchronize()
        except Exception as ex:          # reported by the test
            errors.append(ex)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors
    for t in range(2):
        alone = outputs()
        evaluate(workspaces[t], streams[t], arrays[t], alone)
        streams[t].synchronize()
        results[t] = alone
    return outs, results


def _check(outs, alone):
    for t in range(2):
        for k, o in enumerate(outs[t]):
            for a, b in zip(o, alone[t]):
                assert torch.equal(a, b), (t, k)


def test_two_threads_share_a_plan(M):
    s, other = (inputs.water_box(20001, seed=k, cutoff=12.0, spacing=2.0, order=4) for k in (71, 72))
    plan = M.plan_for(s)
    d = plan.describe()
    print(f"case threads plan layout {d['layout']} short blocks {d['short_blocks']}", flush=True)
    assert d["layout"] == 2
    arrays = [M.to_device(s), M.to_device(other)]
    outs, alone = _run(M, plan, M.lib().msm_compute, M.lib().msm_workspace_init, arrays, s.n, 1, 40)
    _check(outs, alone)
    assert not torch.equal(alone[0][1], alone[1][1])


def test_two_threads_share_a_batch(M):
    systems, other = ([inputs.water_box(n, seed=n + k, cutoff=10.0, spacing=2.0, order=4) for n in (3000, 4500)]
                      for k in (81, 82))
    batch = M.batch_for(systems)
    print("case threads batch", flush=True)
    arrays = [M.batch_to_device(systems), M.batch_to_device(other)]
    outs, alone = _run(M, batch, M.lib().msm_batch_compute, M.lib().msm_batch_workspace_init, arrays, batch.n, 2, 40)
    _check(outs, alone)
