"""Jacobi solves of systems without a value table (nodes off the lattice) on
either side of the size from which an FP64 iteration takes two launches:
stopped after their first iterations against the oracle's conjugate gradients
stopped there too (the iterates are the same in exact arithmetic), and to the
end by the true residual under the oracle's K; and an instance above it in a
batch with others below, bit for bit as on its own."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_1906_08125_amd import workloads as W
from test_gpu_matrix_forms import _moved

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROWS = 400_000


@pytest.fixture(scope="module")
def pic():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_08125_amd import pic as P
    P.load_library()
    return P


def _mesh(nx, ny, nz):
    return _moved(W.kuhn_tip_mesh(nx, ny, nz, 0.5, 2.0, 12.0), 0.08)


@pytest.mark.parametrize("shape,two", [((58, 58, 118), False), ((59, 59, 118), True)])
def test_solve_on_both_sides(pic, shape, two):
    tip = _mesh(*shape)
    om = O.OracleMesh(tip, 10.0)
    gm = pic.Mesh(tip, 10.0)
    assert (gm.n_free > ROWS) == two and abs(gm.n_free - ROWS) < 0.03 * ROWS
    c = np.random.default_rng(5).integers(-2**44, 2**44, tip.n_nodes).astype(np.int64)
    cd = torch.from_numpy(c).cuda()
    for k in (1, 2, 3):
        phi_o, info = om.poisson_solve(c, 1e-3, 0.4, tol=1e-12, max_iter=k)
        phi = torch.zeros(tip.n_nodes, dtype=torch.float64, device="cuda")
        s = gm.solve_stats(gm.poisson_solve(cd, 1e-3, 0.4, phi, tol=1e-12, max_iter=k))
        assert s["iters"] == info["iters"] == k
        assert np.linalg.norm(phi.cpu().numpy() - phi_o) < 1e-9 * np.linalg.norm(phi_o)
    fid, _ = om.free()
    free = np.flatnonzero(fid >= 0)
    free = free[np.argsort(fid[free])]
    b = om.rhs(c, 1e-3, 0.4)
    phi = torch.zeros(tip.n_nodes, dtype=torch.float64, device="cuda")
    for rep in range(2):              # the second replays the captured rounds
        phi.zero_()
        s = gm.solve_stats(gm.poisson_solve(cd, 1e-3, 0.4, phi, tol=1e-10))
        assert s["status"] == 0 and s["relres"] <= 1e-10
        r = b - om.spmv(phi.cpu().numpy()[free])
        assert np.linalg.norm(r) <= 1.5e-10 * np.linalg.norm(b)
    # and in mixed precision after FP64 on the same handle
    phi.zero_()
    s = gm.solve_stats(gm.poisson_solve(cd, 1e-3, 0.4, phi, tol=1e-10,
                                        precision=pic.PIC_MIXED, inner_tol=1e-3))
    assert s["status"] == 0
    r = b - om.spmv(phi.cpu().numpy()[free])
    assert np.linalg.norm(r) <= 1.5e-10 * np.linalg.norm(b)
    gm.close()


def test_two_launch_instance_in_a_batch(pic):
    base = W.config_tiny()
    small = [dataclasses.replace(base, nx=n, ny=n) for n in (12, 14, 16)]
    meshes = [pic.Mesh(c.mesh(), c.emit_zmin) for c in small] + [pic.Mesh(_mesh(62, 62, 126), 10.0)]
    assert meshes[-1].n_free > ROWS
    params = []
    for gm in meshes:
        phi = torch.zeros(gm.n_nodes, dtype=torch.float64, device="cuda")
        E = torch.zeros(4 * gm.n_nodes, dtype=torch.float64, device="cuda")
        gm.poisson_solve(None, 0.0, 0.4, phi, E, tol=1e-9)
        per_run = gm.emission_rate(E, 4.5)[0].item() * 0.5 * 10
        params.append(dict(dt=0.5, E0=0.4, w_sp=0.05 / 3000, phi_w=4.5, seed=7,
                           j_scale=0.05 / per_run, tol=1e-9, resort_every=0))

    def states():
        out = []
        for gm in meshes:
            st = pic.State(gm, 30_000)
            st.init_field(0.4, tol=1e-9)
            out.append(st)
        return out

    single = states()
    ref = [[pic.State.decode_stats(st.step(step0=k, **kw))[0] for k in range(3)]
           for st, kw in zip(single, params)]
    both = states()
    batch = pic.Batch(meshes, both, params)
    for k in range(3):
        sc = batch.schedule()
        for i in range(len(meshes)):
            sc.cg_blocks[i] = int(batch.limits[i][2])
        rows = pic.Batch.decode(batch.step(k, 1, sched=sc), len(meshes))[0]
        for i in range(len(meshes)):
            for key in ("cg_iters", "status", "n_inj", "n_after", "q_after"):
                assert rows[i][key] == ref[i][k][key], (k, i, key)
    for i in range(len(meshes)):
        assert sum(r["cg_iters"] for r in ref[i]) > 20, i
        assert torch.equal(both[i].phi, single[i].phi), i
    batch.close()
    for m in meshes:
        m.close()
