"""The metal solver's row loop where the other tests do not reach: several
slices per wave (more rows than one resident round of workgroups has threads)
against the oracle's matrix, and rows with more entries than one trip takes
against the oracle's solution."""
import numpy as np
import pytest

from oracle import metal as OM
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


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float64)).cuda()


@pytest.mark.parametrize("shape,trips", [((78, 79, 19), 1), ((80, 81, 19), 2), ((113, 114, 19), 3)])
def test_several_slices_per_wave(pic, shape, trips):
    nx, ny, depth = shape
    m = W.kuhn_metal_mesh(nx, ny, 40, 0.5, 2.0, 8.0, depth)
    round_ = 2 * torch.cuda.get_device_properties(0).multi_processor_count * 256
    assert -(-m.n_nodes // round_) == trips, m.n_nodes
    rng = np.random.default_rng(3)
    sigma = 0.5 + 1.5 * rng.random(m.n_tets)
    flux = rng.normal(0.0, 0.2, m.n_faces)
    gm = pic.Metal(m)
    phi, pj, st = gm.continuity_solve(_dev(sigma), _dev(flux), tol=1e-11)
    assert st["converged"] and st["iters"] > 50
    x = phi.cpu().numpy()
    free = m.dirichlet == 0
    assert (x[~free] == 0.0).all()
    K = OM.stiffness(m.xyz, m.tet, sigma)
    f = OM.face_load(m.xyz, m.faces, flux)
    r = (f - K @ x)[free]
    # (the recursive residual is tested to 1e-11; the true one keeps to it up
    # to the rounding of K x, under 1e-12 here)
    assert np.linalg.norm(r) < 2e-11 * np.linalg.norm(f[free])
    gm.close()


def _split_star(m, node):
    """m with the tetrahedra around a node split in four at their centroids:
    the node gains a neighbour per tetrahedron."""
    star = np.flatnonzero((m.tet == node).any(axis=1))
    assert not np.isin(star, m.face_tet).any()
    cen = m.xyz[m.tet[star]].mean(axis=1)
    new = m.n_nodes + np.arange(star.size, dtype=np.int32)
    parts = []
    for k in range(4):
        t = m.tet[star].copy()
        t[:, k] = new
        parts.append(t)
    tet = m.tet.copy()
    tet[star] = parts[0]
    tet = np.ascontiguousarray(np.concatenate([tet] + parts[1:]), np.int32)
    return W.MetalMesh(np.concatenate([m.xyz, cen]), tet, m.faces, m.face_tet,
                       np.concatenate([m.dirichlet, np.zeros(star.size, np.uint8)]),
                       m.z_bottom)


def test_rows_longer_than_a_trip(pic):
    m = W.kuhn_metal_mesh(12, 12, 24, 0.5, 2.0, 6.0, 6)
    z = m.xyz[:, 2]
    inner = np.flatnonzero((z > m.z_bottom + 0.9) & (z < -0.9) &
                           (np.abs(m.xyz[:, 0] - 3.0) < 1.5) & (np.abs(m.xyz[:, 1] - 3.0) < 1.5))
    for node in (inner[0], inner[-1]):
        m = _split_star(m, node)
    rng = np.random.default_rng(4)
    sigma = 0.5 + 1.5 * rng.random(m.n_tets)
    flux = rng.normal(0.0, 0.2, m.n_faces)
    K = OM.stiffness(m.xyz, m.tet, sigma)
    assert np.diff(K.indptr).max() > 32
    want = OM.continuity_solve(m, sigma, flux)
    gm = pic.Metal(m)
    phi, pj, st = gm.continuity_solve(_dev(sigma), _dev(flux), tol=1e-13)
    assert st["converged"]
    x = phi.cpu().numpy()
    assert np.linalg.norm(x - want) < 1e-9 * np.linalg.norm(want)
    pw = OM.joule(m, sigma, want)
    assert np.linalg.norm(pj.cpu().numpy() - pw) < 1e-9 * np.linalg.norm(pw)
    gm.close()
