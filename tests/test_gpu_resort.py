"""The re-sort against numpy's stable sort of the same slots: at the edge
between the tile counts that the scatter sums and those of a scan launch
(64 tiles of 4,096 slots), with two and three digit passes, ragged and empty
populations, alone and in a batch whose instances differ in all of these and
are not all due."""
import numpy as np
import pytest

from paper_1906_08125_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ARRAYS = ("x", "y", "z", "vx", "vy", "vz", "w", "tet", "birth", "id")


@pytest.fixture(scope="module")
def pic():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_08125_amd import pic as P
    P.load_library()
    return P


def _held(gm, n, seed):
    """n injected particles spread at random over the emitting faces."""
    held = np.zeros(gm.n_emit, np.int32)
    np.add.at(held, np.random.default_rng(seed).integers(0, gm.n_emit, n), 1)
    return torch.from_numpy(held).cuda()


def _slots(gs):
    n = int(gs.n_slots.item())
    return {k: getattr(gs, k)[:n].cpu().numpy() for k in ARRAYS}


def _sorted(A):
    """What a re-sort leaves of the slots A."""
    live = np.flatnonzero(A["tet"] >= 0)
    order = live[np.argsort(A["tet"][live], kind="stable")]
    return {k: A[k][order] for k in ARRAYS}


# (three digits, capacity, injected)
CASES = [(False, 64 * 4096, 4096), (False, 64 * 4096 + 1, 4097), (True, 20_000, 12_289),
         (True, 65 * 4096, 70_001), (False, 4096, 0), (True, 5_000, 63)]


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("batched", [False, True])
def test_resort_is_a_stable_sort_of_the_live_slots(pic, batched, mixed):
    tiny = W.config_tiny()
    big = W.batch_configs(1)[0]
    mesh = {}
    runs = []
    for every in (0, 2):
        meshes, states, params = [], [], []
        for i, (three, cap, n_inj) in enumerate(CASES):
            cfg = big if three else tiny
            # a mesh of its own per instance of the batch
            gm = mesh.get(i) or pic.Mesh(cfg.mesh(), cfg.emit_zmin)
            mesh[i] = gm
            assert (gm.n_tets >= 1 << 16) == three
            gs = pic.State(gm, cap, precision=pic.PIC_MIXED if mixed else pic.PIC_FP64)
            gs.init_field(cfg.E0, tol=cfg.tol)
            meshes.append(gm)
            states.append(gs)
            # (the last instance of a batch is not due in these steps)
            params.append(dict(dt=cfg.dt, E0=cfg.E0, w_sp=1e-9, phi_w=cfg.phi_w,
                               seed=cfg.seed, tol=cfg.tol,
                               resort_every=5 if every and i == len(CASES) - 1 else every,
                               counts_in=_held(gm, n_inj, i)))
        for k in range(2):
            if k:
                for p, (_, _, n_inj), gm in zip(params, CASES, meshes):
                    p["counts_in"] = _held(gm, 0, 0)
            if batched:
                rows = pic.Batch.decode(pic.Batch(meshes, states, params).step(k, 1),
                                        len(CASES))[0]
            else:
                rows = [pic.State.decode_stats(gs.step(step0=k, **p))[0]
                        for gs, p in zip(states, params)]
        torch.cuda.synchronize()
        runs.append(([_slots(gs) for gs in states], rows))
    (plain, _), (sort, rows) = runs
    for i, (three, cap, n_inj) in enumerate(CASES):
        want = plain[i] if i == len(CASES) - 1 else _sorted(plain[i])
        assert rows[i]["n_slots"] == want["id"].size, i
        for k in ARRAYS:
            assert (sort[i][k] == want[k]).all(), (i, k)
        if n_inj > 4096:
            assert want["id"].size > 3000, i
