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


# The particle step by domain blocks: one block, two and several (odd cuts,
# one-cell-wide remainders impossible to avoid), flights that cross many of
# them and end on every wall, with and without face tallies, null collisions,
# expected-value rays; more flights than one unit of work takes.
BLOCKS = {
    "null_one_block": (lambda: two_material_2d(n=61, kn_right=0.05, ratio=30.0, particles=300_000), {}),
    "null_wide": (lambda: _two_tau(301, 71, 0.02, 0.5, 400_000), {}),
    "null_tall": (lambda: _two_tau(67, 290, 0.02, 1.0, 400_000), {}),
    "null_many": (lambda: _two_tau(211, 197, 0.004, 0.4, 300_000), {}),
    "ev_one_block": (lambda: cavity_2d(n=90, ny=77, kn=0.3, particles=220_000, newton=False), {"estimator": 1}),
    "ev_many": (lambda: cavity_2d(n=230, ny=170, kn=0.2, particles=220_000, newton=False), {"estimator": 1}),
    "null_few_flights": (lambda: _two_tau(70, 61, 0.2, 0.9, 37_000), {}),
    "null_no_weight": (lambda: _two_tau(101, 90, 0.1, 0.5, 60_000), {"T_init": "ref"}),
    "ev_null": (lambda: _two_tau(150, 141, 0.05, 0.5, 220_000), {"estimator": 1}),
}


def _two_tau(nx, ny, kn_a, kn_b, particles):
    """A cavity with two relaxation times in an irregular pattern."""
    w = cavity_2d(n=nx, ny=ny, kn=kn_a, particles=particles, newton=False)
    w.tau = np.where(np.random.default_rng(5).random(w.n_cells) < 0.5, kn_a, kn_b)
    return w


@pytest.mark.parametrize("name", list(BLOCKS))
@pytest.mark.parametrize("faces", [True, False])
def test_domain_blocks_bitwise(oracle_mod, gpu, name, faces):
    make, kw = BLOCKS[name]
    w = make()
    mode = oracle_mod.FACES_EVERY if faces else oracle_mod.FACES_OFF
    kw = dict({"T_init": seeded_temperature(w.n_cells)}, **kw)
    if isinstance(kw["T_init"], str):       # (only the walls emit at first)
        kw["T_init"] = np.full(w.n_cells, w.t_ref)
    o, s = _pair(oracle_mod, gpu, w, tally_faces=mode, **kw)
    for i in range(2):
        assert o.step(1) == 0 and s.step(1) == 0
        if faces:
            _same_iteration(o, s, f"{name} it{i}")
        else:
            _same_cells(o, s, f"{name} it{i}")


@pytest.mark.parametrize("faces", [True, False])
def test_domain_blocks_bands_bitwise(oracle_mod, gpu, faces):
    """Three bands in one launch, one of them without null collisions, several
    blocks each: domain blocks (march 0) against every band on tiles."""
    from synth import nongray_two_material_2d
    w = nongray_two_material_2d(n=120, K=3, ratio=20.0, particles=400_000)
    w.tau = w.tau.copy()
    w.tau[120 * 120: 2 * 120 * 120] = w.tau[-1]
    mode = gpu.FACES_EVERY if faces else gpu.FACES_OFF
    T0 = seeded_temperature(w.n_cells)
    a = gpu.Solver(w, tally_faces=mode, T_init=T0)
    b = gpu.Solver(w, tally_faces=mode, T_init=T0, march=1)
    for it in range(2):
        assert a.step(1) == 0 and b.step(1) == 0
        ta, tb = a.tallies(), b.tallies()
        for k in ta if faces else ("D", "W", "B"):
            assert torch.equal(ta[k], tb[k]), (it, k)
        assert torch.equal(a.state()[2], b.state()[2]) and torch.equal(a.state()[3], b.state()[3])
    sa, sb = a.stats(), b.stats()
    for k in ("flights", "segments", "crossings"):
        assert sa[k] == sb[k]


# The multigrid-preconditioned CG: levels in LDS with records (at most one cell
# per thread and six levels below the first) and without, a first LDS level of
# one, two and many cells per thread, groups on one XCD and device-wide, more
# members than rows, windows of one row, rows too long for the windows beside
# the LDS levels or for any; odd sizes at each level; and operators so large
# that no reciprocal is used in place of a division.
MG = {
    "lds_32x32": (32, 32, 0, 1.0), "lds_33x31": (33, 31, 0, 1.0), "lds_33x31_w1": (33, 31, 1, 1.0),
    "lds_2x500": (2, 500, 0, 1.0), "lds_500x2": (500, 2, 0, 1.0), "lds_5x1": (5, 1, 0, 1.0),
    "xcd_33x32": (33, 32, 0, 1.0), "xcd_65x63_w2": (65, 63, 2, 1.0), "xcd_129x127": (129, 127, 0, 1.0),
    "device_257x255": (257, 255, 0, 1.0), "tall_9x1200": (9, 1200, 0, 1.0),
    "wide_700x9": (700, 9, 0, 1.0), "wide_790x30": (790, 30, 0, 1.0), "wide_1500x5": (1500, 5, 0, 1.0),
    "huge_40x36": (40, 36, 0, 1e95), "huge_30x20": (30, 20, 0, 1e95),
}


@pytest.mark.parametrize("name", list(MG))
def test_mg_launch_forms_bitwise(oracle_mod, gpu, name):
    nx, ny, waves, scale = MG[name]
    w = cavity_2d(n=nx, ny=ny, kn=0.02, particles=20 * nx * ny)
    rng = np.random.default_rng(nx * ny)
    D = rng.uniform(0.5, 2.0, size=(2, w.n_cells)) * w.vg * 1e-2 * scale
    kw = dict(newton=True, diff_x=D[0], diff_y=D[1], tally_faces=oracle_mod.FACES_OFF,
              cg_precond=oracle_mod.PRECOND_MG, T_init=seeded_temperature(w.n_cells))
    o = oracle_mod.Oracle(w, **kw)
    s = gpu.Solver(w, cg_waves=waves, **kw)
    for i in range(2):
        assert o.step(1) == 0 and s.step(1) == 0
        _, _, E, G = s.state()
        assert np.array_equal(o.E(), E.cpu().numpy()), f"{name} iteration {i}: E differs"
        assert np.array_equal(o.G(), G.cpu().numpy()), f"{name} iteration {i}: G differs"
        assert o.info().cg_iters_last == s.stats()["cg_iters_last"], name


@pytest.mark.parametrize("nx,ny", [(5, 1), (40, 36), (131, 129)])
def test_emission_budget_overflow_status(oracle_mod, gpu, nx, ny):
    """A Newton step whose emission leaves the fixed-point range (a group velocity
    of 1e-96 under the same residual) reports what the oracle reports, with one
    partial sum of the budget and with several per thread."""
    w = cavity_2d(n=nx, ny=ny, kn=0.02, particles=20 * nx * ny)
    rng = np.random.default_rng(nx * ny)
    w.vg *= 1e-96
    w.tau = w.tau / 1e-96
    D = rng.uniform(0.5, 2.0, size=(2, w.n_cells)) * w.vg * 1e-2
    kw = dict(newton=True, diff_x=D[0], diff_y=D[1], tally_faces=oracle_mod.FACES_OFF,
              cg_precond=oracle_mod.PRECOND_MG, T_init=seeded_temperature(w.n_cells))
    o = oracle_mod.Oracle(w, **kw)
    s = gpu.Solver(w, **kw)
    rc = o.step(1)
    assert rc != 0 and s.step(1) == rc


@pytest.mark.parametrize("n", [128, 256])
def test_mg_groups_of_many_streams(gpu, oracle_mod, n):
    """Newton steps with the multigrid CG from eight threads at once, each on a
    stream of its own: what each solver returns alone."""
    import threading

    w = cavity_2d(n=n, kn=0.1, particles=100_000, newton=True)
    kw = dict(tally_faces=oracle_mod.FACES_OFF, cg_precond=gpu.PRECOND_MG, own_stream=True)
    one = gpu.Solver(w, **kw)
    for _ in range(3):
        assert one.step(1) == 0
    ss = [gpu.Solver(w, **kw) for _ in range(8)]
    rcs = [None] * 8

    def work(i):
        rcs[i] = [ss[i].step(1) for _ in range(3)]

    ts = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for s, rc in zip(ss, rcs):
        assert rc == [0, 0, 0]
        assert torch.equal(s.state()[2], one.state()[2])
