"""Two batches stepped by two threads on streams of their own, each with more
injecting workgroups than fit on the chip at once (all of which wait for the
emission of their instance): each as the same batch on its own, to the bit."""
import threading

import pytest

from paper_1906_08125_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N_INST, STEPS, CALLS = 4, 5, 4


def _batch(pic, first):
    cfg = W.config_tiny()
    meshes, states, params = [], [], []
    for i in range(first, first + N_INST):
        gm = pic.Mesh(cfg.mesh(), 0.5)
        gs = pic.State(gm, 60_000)
        gs.init_field(cfg.E0, tol=cfg.tol)
        rate, _ = gm.emission_rate(gs.E, cfg.phi_w)
        w_sp = rate.item() * cfg.dt / 500
        meshes.append(gm)
        states.append(gs)
        params.append(dict(dt=cfg.dt, E0=cfg.E0, w_sp=w_sp, phi_w=cfg.phi_w, seed=3 + i,
                           tol=cfg.tol, resort_every=4))
    return pic.Batch(meshes, states, params)


def _run(pic, b, out):
    for c in range(CALLS):
        sc = b.schedule()
        for i in range(N_INST):
            sc.inject_blocks[i] = int(b.limits[i][1])
        out += [r for k in pic.Batch.decode(b.step(c * STEPS, STEPS, sched=sc), N_INST) for r in k]


def test_batches_of_two_streams():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_08125_amd import pic
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    alone, rows = [], []
    for first in (0, N_INST):
        b = _batch(pic, first)
        assert sum(int(b.limits[i][1]) for i in range(N_INST)) > 4 * cus
        rows.append([])
        _run(pic, b, rows[-1])
        torch.cuda.synchronize()
        alone.append([(s.x.clone(), s.tet.clone(), s.phi.clone()) for s in b.states])
        b.close()
    both = [_batch(pic, first) for first in (0, N_INST)]
    torch.cuda.synchronize()
    got, errors = [[], []], []

    def work(j):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                _run(pic, both[j], got[j])
                torch.cuda.current_stream().synchronize()
        except Exception as e:      # (reported below: a thread's own are lost)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(j,)) for j in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for j in range(2):
        assert all(r["status"] == 0 for r in got[j])
        assert sum(r["n_inj"] for r in got[j]) > 10_000
        assert got[j] == rows[j]
        for s, (x, tet, phi) in zip(both[j].states, alone[j]):
            n = int(s.n_slots.item())
            assert torch.equal(s.x[:n], x[:n]) and torch.equal(s.tet[:n], tet[:n])
            assert torch.equal(s.phi, phi)
    for b in both:
        b.close()
