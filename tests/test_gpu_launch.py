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


def _same_cells(o, s, tag):
    to, ts = o.tallies(), s.tallies()
    for k in ("D", "W", "B"):
        assert np.array_equal(to[k], ts[k].cpu().numpy()), f"{tag} tally {k} differs"
    _, _, E, G = s.state()
    assert np.array_equal(o.E(), E.cpu().numpy()) and np.array_equal(o.G(), G.cpu().numpy()), tag
    oi, st = o.info(), s.stats()
    assert (oi.flights, oi.segments, oi.crossings) == (st["flights"], st["segments"], st["crossings"])


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
        if faces:
            _same_iteration(o, s, f"{name} it{i}")
        else:                       # (no face fluxes to compare)
            _same_cells(o, s, f"{name} it{i}")


# The diffusion correction's linear solver in each of its launch forms: one
# workgroup (up to 8 blocks of 256 cells), a group within one XCD (a ragged
# last block, a last workgroup with fewer blocks, halo rows longer than a
# workgroup's range, block sums loaded directly and by shares), a device-wide
# group (more than 256 blocks), the global-memory form (long rows).
CG = {
    "one_2048": (2, 64, 32), "one_1d": (1, 1999, 1), "xcd_2049": (2, 683, 3),
    "xcd_ragged": (2, 101, 67), "xcd_long_rows": (2, 1400, 9), "xcd_1d": (1, 5000, 1),
    "xcd_share": (2, 130, 131), "xcd_256": (2, 257, 255), "device_257": (2, 257, 257),
    "global": (2, 3001, 3),
}


@pytest.mark.parametrize("name", list(CG))
def test_cg_launch_forms_bitwise(oracle_mod, gpu, name):
    dim, nx, ny = CG[name]
    w = slab_1d(n=nx, kn=0.1) if dim == 1 else cavity_2d(n=nx, ny=ny, kn=0.1)
    rng = np.random.default_rng(nx * ny)
    w.tau = w.tau * rng.uniform(0.5, 2.0, size=w.tau.size)
    D = rng.uniform(0.5, 2.0, size=(2, w.tau.size)) * 1e-4
    b = rng.normal(size=w.tau.size)
    its = 60                        # (a prefix of the solve: the last iterate is compared)
    rc_o, x_o, its_o = oracle_mod.cg(w, D[0], D[1] if dim == 2 else None, b, tol=1e-12, max_iters=its)
    for _ in range(2):              # (twice: the scratch of the first call is not the second's)
        rc, x, its_g = gpu.diffusion_solve(w, D[0], D[1], b, tol=1e-12, max_iters=its)
        assert (rc, its_g) == (rc_o, its_o)
        assert np.array_equal(x.cpu().numpy(), x_o)


def test_cg_groups_of_many_streams(gpu):
    """Solves on eight streams from eight threads at once: each group finds its
    workgroups (on one XCD or anywhere) and returns what it returns alone."""
    import threading

    w = cavity_2d(n=256, kn=0.1)
    rng = np.random.default_rng(3)
    D = torch.from_numpy(rng.uniform(0.5, 2.0, size=(2, w.tau.size)) * 1e-4).cuda()
    bs = [torch.from_numpy(rng.normal(size=w.tau.size)).cuda() for _ in range(8)]
    alone = [gpu.diffusion_solve(w, D[0], D[1], b, tol=1e-12, max_iters=200)[1].clone() for b in bs]
    got = [None] * 8

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                got[i] = gpu.diffusion_solve(w, D[0], D[1], bs[i], tol=1e-12, max_iters=200)[1].clone()
            torch.cuda.current_stream().synchronize()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for a, g in zip(alone, got):
        assert torch.equal(a, g)
