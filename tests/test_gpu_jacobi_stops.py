"""A Jacobi solve stopped after each of its first iterations, odd and even (an
even one leaves its share of x to the odd one, or to the pass that ends the
recursion), against the oracle's conjugate gradients stopped there too.  The
iterates are the same in exact arithmetic; in FP64 the bound is the
potential's 1e-9, in mixed precision 2^-24 grown by the condition of a small
system, under 1e-4.  A lost update would show as 1e-2 or more."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1906_08125_amd import workloads as W
from test_gpu_matrix_forms import _moved

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("packed", [True, False])
def test_jacobi_stopped_early(packed):
    from paper_1906_08125_amd import pic
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tip = W.kuhn_tip_mesh(13, 11, 19, 0.5, 1.0, 3.0)
    if not packed:
        tip = _moved(tip, 0.1)
    om = O.OracleMesh(tip, 0.01)
    gm = pic.Mesh(tip, 0.01)
    c = np.random.default_rng(5).integers(-2**44, 2**44, tip.n_nodes).astype(np.int64)
    cd = torch.from_numpy(c).cuda()
    last = None
    for k in range(1, 8):
        phi_o, info = om.poisson_solve(c, 1e-3, 0.4, tol=1e-12, max_iter=k)
        assert info["iters"] == k
        if last is not None:
            assert np.linalg.norm(phi_o - last) > 1e-3 * np.linalg.norm(phi_o)
        last = phi_o
        for prec, bound in ((pic.PIC_FP64, 1e-9), (pic.PIC_MIXED, 1e-4)):
            phi = torch.zeros(tip.n_nodes, dtype=torch.float64, device="cuda")
            s = gm.solve_stats(gm.poisson_solve(cd, 1e-3, 0.4, phi, tol=1e-12, max_iter=k,
                                                precision=prec, inner_tol=1e-7))
            assert s["iters"] == k
            p = phi.cpu().numpy()
            assert np.linalg.norm(p - phi_o) < bound * np.linalg.norm(phi_o), (k, prec)
    gm.close()
