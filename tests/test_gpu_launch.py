"""Launch forms of the kernels at the sizes where they can go wrong, bit for bit
against the oracle (integer tallies and the same IEEE operations in the same
order: no tolerance)."""
import numpy as np
import pytest

from synth import cavity_2d, seeded_temperature, slab_1d, slab_1d_two_tau, two_material_2d
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


# A tile's particles split over several workgroups: one cell with many
# particles (one workgroup's share below a wavefront at the end), remainders in
# every part, null collisions with and without lane refill, one particle per
# emitter (no split), a 1D mesh beyond and within the whole-domain window.
SPLIT = {
    "one_cell": lambda: slab_1d(n=1, kn=0.5, particles=100_003),
    "slab_17": lambda: slab_1d(n=17, kn=0.3, particles=300_007),
    "slab_17_two_tau": lambda: slab_1d_two_tau(n=17, particles=300_007),
    "slab_one_each": lambda: slab_1d(n=300, kn=0.3, particles=302),
    "slab_window": lambda: slab_1d_two_tau(n=3300, tau_left=0.1, tau_right=0.001, particles=60_000),
    "slab_whole": lambda: slab_1d_two_tau(n=1500, tau_left=0.1, tau_right=0.001, particles=60_000),
    "ragged_19x13": lambda: cavity_2d(n=19, ny=13, kn=0.2, particles=200_003, newton=False),
    "null_26": lambda: two_material_2d(n=26, kn_right=0.05, ratio=30.0, particles=300_011),
}


@pytest.mark.parametrize("name", sorted(SPLIT))
@pytest.mark.parametrize("faces", [True, False])
def test_split_tiles_bitwise(oracle_mod, gpu, name, faces):
    w = SPLIT[name]()
    mode = oracle_mod.FACES_EVERY if faces else oracle_mod.FACES_OFF
    o, s = _pair(oracle_mod, gpu, w, tally_faces=mode, T_init=seeded_temperature(w.n_cells),
                 march=1)
    for i in range(2):
        assert o.step(1) == 0 and s.step(1) == 0
        _same_iteration(o, s, f"{name} it{i}")
