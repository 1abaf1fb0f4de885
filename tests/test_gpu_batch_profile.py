"""Kernel timing of batched steps: every class counts what a step does once,
whichever instances' particle kernels ran ahead of their solve, were held back
by it or launched again."""
import pytest

from paper_1906_08125_amd import workloads as W
from test_gpu_batch import _cases, _setup
from test_gpu_matrix_forms import _moved

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pic():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_08125_amd import pic as P
    P.load_library()
    return P


# charge in flight of each instance (1e-15: no solve iterates); general: the
# middle one off the lattice, so that it has other tet records
@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("live", [(1e-15, 1e-15, 1e-15), (0.01, 1e-15, 0.01), (0.01, 0.01, 0.01),
                                  (1e-15, 0.01, 1e-15)])
def test_batch_counts(pic, live, general):
    cap, warm, steps = 20_000, 4, 6
    cases = [_setup(pic, c, q, 3000, cap) for c, q in zip(_cases(), live)]
    meshes = [c[3] for c in cases]
    if general:
        meshes[1] = pic.Mesh(_moved(cases[1][0], 0.08), _cases()[1].emit_zmin)
    states, params = [], []
    for gm, (tip, om, ost, _, kw) in zip(meshes, cases):
        gs = pic.State(gm, cap)
        gs.init_field(kw["E0"], tol=kw["tol"])
        states.append(gs)
        params.append(dict(kw, resort_every=5))
    batch = pic.Batch(meshes, states, params)
    batch.step(0, warm)
    meshes[0].profile(True)
    rows = pic.Batch.decode(batch.step(warm, steps), len(cases))
    kt = meshes[0].profile_read()
    meshes[0].profile(False)
    iterated = [sum(r[i]["cg_iters"] for r in rows) > 0 for i in range(len(cases))]
    assert iterated == [q > 1e-3 for q in live]
    # (instances with and without packed records have a launch each)
    want = dict(push=steps * (2 if general else 1), emit=1, fallback=steps, solve=steps, sort=2)
    for k, n in want.items():
        assert kt[k]["launches"] == n, (k, kt)
        assert kt[k]["ms"] > 0.0
