"""The particle kernels on the two forms of the tet records against the
oracle: packed (few distinct barycentric maps: the lattice) and full (nodes
off the lattice), in every storage precision and field mode, with the walk,
the exact fallback and the stand-alone location."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_1906_08125_amd import workloads as W
from test_gpu_matrix_forms import _moved
from test_gpu_parity import _compare_mixed, _compare_runs, _run_pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pic():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_08125_amd import pic as P
    P.load_library()
    return P


@dataclasses.dataclass
class _Cfg(W.RunConfig):
    moved: float = 0.0

    def mesh(self):
        m = super().mesh()
        return _moved(m, self.moved) if self.moved else m


def _config(form):
    c = dataclasses.asdict(W.config_tiny())
    return _Cfg(**c, moved=0.08 if form == "full" else 0.0)


@pytest.mark.parametrize("field_mode", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("form", ["packed", "full"])
def test_steps(pic, form, precision, field_mode):
    cfg = _config(form)
    err = []
    _, ost, _, gs, so, sg = _run_pair(pic, cfg, 9, 0.01, 3000, 60_000, resort_every=4,
                                      precision=precision, field_mode=field_mode,
                                      phi_err=err)
    assert sum(s["n_inj"] for s in sg) > 500
    if precision:
        _compare_mixed(ost, gs, so, sg, err)
    else:
        _compare_runs(ost, gs, so, sg)


@pytest.mark.parametrize("hint", [False, True])
@pytest.mark.parametrize("n", [1, 63, 257, 20_000])
@pytest.mark.parametrize("form", ["packed", "full"])
def test_locate(pic, form, n, hint):
    """Points anywhere in the box and past the anode, with hints far off or
    none: the canonical tet, bit for bit, in both location calls."""
    tip = _config(form).mesh()
    om = O.OracleMesh(tip, 0.01)
    gm = pic.Mesh(tip, 0.01)
    p = W.random_points_in_box(tip, n, 5)
    p[:, 2] *= 1.02
    g = np.random.default_rng(1)
    h = g.integers(0, tip.n_tets, n).astype(np.int32) if hint else np.full(n, -1, np.int32)
    if hint:
        h[::3] = tip.n_tets + 5       # out of range: as none
    t_o, w_o = om.locate(p, np.full(n, -1, np.int32))
    x, y, z = (torch.from_numpy(np.ascontiguousarray(p[:, k])).cuda() for k in range(3))
    for call in (gm.locate, gm.locate_noalloc):
        tet = torch.from_numpy(h.copy()).cuda()
        where = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
        call(x, y, z, tet, where)
        assert (tet.cpu().numpy() == t_o).all()
        assert (where.cpu().numpy() == w_o).all()
    gm.close()
