"""A batched call of several steps, whose particle launches run ahead of the
solves, against the oracle: instances whose solves end at once, after a
speculated round or after several, under either preconditioner, so that in
every step some are let through and others launched again; re-sorts of their
own period, some of them never."""
import pytest

from test_gpu_batch import _cases, _setup
from test_gpu_parity import _compare_runs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pic():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_08125_amd import pic as P
    P.load_library()
    return P


# charge in flight of each instance (1e-15: no solve iterates)
@pytest.mark.parametrize("live", [(1e-15, 0.01, 1e-15), (0.01, 1e-15, 0.01), (0.01, 0.01, 0.01)])
@pytest.mark.parametrize("amg", [False, True])
def test_batch_steps_ahead_match_oracle(pic, live, amg):
    cap, calls = 20_000, (1, 4, 3)
    cases = [_setup(pic, c, q, 3000, cap) for c, q in zip(_cases(), live)]
    states, params = [], []
    for i, (tip, om, ost, gm, kw) in enumerate(cases):
        pre = pic.PIC_PRECOND_AMG if amg and i != 1 else pic.PIC_PRECOND_JACOBI
        gs = pic.State(gm, cap, precond=pre)
        gs.init_field(kw["E0"], tol=kw["tol"])
        states.append(gs)
        params.append(dict(kw, resort_every=(2, 3, 0)[i]))
    batch = pic.Batch([c[3] for c in cases], states, params)
    so = [[] for _ in cases]
    sg = [[] for _ in cases]
    k0 = 0
    for n in calls:
        for row in pic.Batch.decode(batch.step(k0, n), len(cases)):
            for i in range(len(cases)):
                sg[i].append(row[i])
        for k in range(k0, k0 + n):
            for i, (tip, om, ost, gm, kw) in enumerate(cases):
                so[i].append(ost.step(step=k, **kw))
        k0 += n
    torch.cuda.synchronize()
    for i, (tip, om, ost, gm, kw) in enumerate(cases):
        assert (sum(s["cg_iters"] for s in sg[i][1:]) > 0) == (live[i] > 1e-3), i
        _compare_runs(ost, states[i], so[i], sg[i], same_solver=not (amg and i != 1))
