"""The domain blocks' place among the particle step's forms: which iterations
take them, and that every form a handle chooses gives the oracle's tallies bit
for bit (integer tallies and the same IEEE operations in the same order: no
tolerance)."""
import pytest

from synth import cavity_2d, nongray_two_material_2d, seeded_temperature, two_material_2d
from test_gpu_bands import _same_state
from test_gpu_parity import _pair, _same_iteration

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_09465_amd as P
    P.library()
    return P


# Handles without face tallies whose iterations run by domain blocks, asked for
# an iteration with them (iugkp_step_faces): its y-face tallies have to be kept
# somewhere.
FACES_ON_DEMAND = {
    "rays": (lambda: cavity_2d(n=60, ny=47, kn=0.3, particles=90_000, newton=False), {"estimator": 1}),
    "rays_null": (lambda: two_material_2d(n=50, kn_right=0.1, ratio=10.0, particles=60_000),
                  {"estimator": 1}),
    "null": (lambda: two_material_2d(n=61, kn_right=0.05, ratio=30.0, particles=300_000), {}),
}


@pytest.mark.parametrize("name", list(FACES_ON_DEMAND))
def test_faces_on_demand_without_face_tallies(oracle_mod, gpu, name):
    make, kw = FACES_ON_DEMAND[name]
    w = make()
    o, s = _pair(oracle_mod, gpu, w, tally_faces=oracle_mod.FACES_OFF,
                 T_init=seeded_temperature(w.n_cells), **kw)
    for faces in (False, True, False, True):
        assert o.step(1, faces=faces) == 0 and s.step(1, faces=faces) == 0
        if faces:
            _same_iteration(o, s, name)


def test_faces_on_demand_without_face_tallies_bands(oracle_mod, gpu):
    w = nongray_two_material_2d(n=48, K=3, ratio=20.0, particles=150_000)
    o = oracle_mod.Bands(w, tally_faces=oracle_mod.FACES_OFF)
    s = gpu.Solver(w, tally_faces=gpu.FACES_OFF)
    for i, faces in enumerate((False, True, False, True)):
        assert o.step(1, faces=faces) == 0 and s.step(1, faces=faces) == 0
        if faces:
            _same_state(o, s, f"it{i}")
