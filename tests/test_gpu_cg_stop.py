"""Jacobi solves of many instances in shared launches, with far more
workgroups than are resident at once: the late ones start while workgroup 0
may already have stopped the recursion, and all of a workgroup's waves have
to take the same way.  With the solver grid that a handle uses by itself the
sums are split alike, so the potentials are those of the same instances
stepped one by one, bit for bit, and so are the iteration counts."""
import pytest

from paper_1906_08125_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N_INST, CAP, STEPS = 8, 30_000, 6


def _config(i):
    return W.RunConfig(f"tip_{i}", 20 + i, 20, 40, 0.5, 2.0, 8.0, 0.4 + 0.02 * i, 4.5, 0.5, 10,
                       1e-12, 3000, 0.01, 3 + i, 0, 8)


@pytest.mark.parametrize("precision", [0, 1])
def test_late_workgroups_stop_alike(precision):
    from paper_1906_08125_amd import pic
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfgs = [_config(i) for i in range(N_INST)]
    meshes = [pic.Mesh(c.mesh(), c.emit_zmin) for c in cfgs]
    params = []
    for c, gm in zip(cfgs, meshes):
        phi = torch.zeros(gm.n_nodes, dtype=torch.float64, device="cuda")
        E = torch.zeros(4 * gm.n_nodes, dtype=torch.float64, device="cuda")
        gm.poisson_solve(None, 0.0, c.E0, phi, E, tol=c.tol)
        per_run = gm.emission_rate(E, c.phi_w)[0].item() * c.dt * c.transit_steps
        scale = 0.05 / per_run          # electrons in flight: every solve iterates
        params.append(dict(dt=c.dt, E0=c.E0, w_sp=0.05 / 3000, phi_w=c.phi_w, seed=c.seed,
                           j_scale=scale, tol=1e-11, resort_every=0))

    def states():
        out = []
        for c, gm in zip(cfgs, meshes):
            st = pic.State(gm, CAP, precision=precision)
            st.init_field(c.E0, tol=1e-11)
            out.append(st)
        return out

    # one by one
    single = states()
    ref = []
    for st, kw in zip(single, params):
        ref.append([pic.State.decode_stats(st.step(step0=k, **kw))[0] for k in range(STEPS)])
    # together, every instance with its handle's own solver grid
    both = states()
    batch = pic.Batch(meshes, both, params)
    blocks = 0
    for k in range(STEPS):
        sc = batch.schedule()
        blocks = 0
        for i in range(N_INST):
            sc.cg_blocks[i] = int(batch.limits[i][2])
            blocks += sc.cg_blocks[i]
        rows = pic.Batch.decode(batch.step(k, 1, sched=sc), N_INST)[0]
        for i in range(N_INST):
            for key in ("cg_iters", "status", "n_inj", "n_after", "q_after"):
                assert rows[i][key] == ref[i][k][key], (k, i, key)
            assert rows[i]["status"] == 0
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert blocks > 2 * 2 * cus         # (512 threads: two resident per CU)
    assert all(sum(r["cg_iters"] for r in rows) > 20 for rows in ref)
    for i in range(N_INST):
        assert torch.equal(both[i].phi, single[i].phi), i
        assert torch.equal(both[i].E, single[i].E), i
    batch.close()
    for m in meshes:
        m.close()
