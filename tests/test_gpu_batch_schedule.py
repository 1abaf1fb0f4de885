"""The workgroup counts of a batch: a call launches those that its schedule
asks for, and the Python side's own schedule fills the chip."""
import pytest

from paper_1906_08125_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pic():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_08125_amd import pic as P
    P.load_library()
    return P


def _batch(pic, n_particles):
    cfg = W.config_tiny()
    meshes, states, params = [], [], []
    for i in range(2):
        gm = pic.Mesh(cfg.mesh(), cfg.emit_zmin)
        gs = pic.State(gm, 4 * n_particles)
        gs.init_field(cfg.E0, tol=cfg.tol)
        rate, _ = gm.emission_rate(gs.E, cfg.phi_w)
        w_sp = rate.item() * cfg.dt * cfg.transit_steps / n_particles
        meshes.append(gm)
        states.append(gs)
        params.append(dict(dt=cfg.dt, E0=cfg.E0, w_sp=w_sp, phi_w=cfg.phi_w, seed=3 + i,
                           tol=cfg.tol, resort_every=10))
    return pic.Batch(meshes, states, params)


def test_a_schedule_is_kept(pic):
    """Eight push workgroups are eight (a few dozen superparticles per thread
    one after another), and the results do not depend on the counts."""
    ms, out = {}, {}
    for blocks in (8, 512):
        b = _batch(pic, 200_000)
        b.step(0, 20)
        b.meshes[0].profile(True, classes=("push",))
        for k in range(5):
            sc = b.schedule()
            for i in range(2):
                sc.push_blocks[i] = blocks
            b.step(20 + k, 1, sched=sc)
        ms[blocks] = b.meshes[0].profile_read()["push"]["ms"]
        b.meshes[0].profile(False)
        torch.cuda.synchronize()
        out[blocks] = [(s.x.clone(), s.tet.clone(), s.charge.clone()) for s in b.states]
        n = [int(s.n_slots.item()) for s in b.states]
        assert min(n) > 100_000
        b.close()
    assert ms[8] > 2.0 * ms[512], ms
    for A, B, m in zip(out[8], out[512], n):
        assert torch.equal(A[0][:m], B[0][:m]) and torch.equal(A[1][:m], B[1][:m])
        assert torch.equal(A[2], B[2])


@pytest.mark.parametrize("tile", [None, 1024, 8192])
def test_own_schedule_fills_the_chip(pic, tile):
    b = _batch(pic, 30_000)
    b.step(0, 10)
    sc = b.schedule(push_tile=tile)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    push = sum(sc.push_blocks[i] for i in range(2))
    inj = sum(sc.inject_blocks[i] for i in range(2))
    # one resident round of four per CU, the emitting workgroups included
    assert 4 * cus - 8 - 16 <= push + inj + 8 <= 4 * cus
    for i in range(2):
        assert sc.push_blocks[i] % 8 == 0 and sc.push_blocks[i] <= b.limits[i][0]
    b.close()
