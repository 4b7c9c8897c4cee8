"""The domain blocks' place among the particle step's forms: which iterations
take them, and that every form a handle chooses gives the oracle's tallies bit
for bit (integer tallies and the same IEEE operations in the same order: no
tolerance)."""
import numpy as np
import pytest

from synth import cavity_2d, nongray_two_material_2d, seeded_temperature, two_material_2d
from test_gpu_bands import _same_state
from test_gpu_launch import BLOCKS, _same_cells
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


def _settle(s, most=8):
    for _ in range(most):
        if s.march_tuning()[0] is not None:
            return
        assert s.step(1) == 0
    assert s.march_tuning()[0] is not None


@pytest.mark.parametrize("n,first,second", [(61, 3.0, 100.0), (63, 100.0, 3.0)])
def test_a_measured_form_holds_for_its_own_class(gpu, n, first, second):
    """Two problems that differ only in the ratio of their relaxation times: at 3
    flights stay near and blocks are no candidate, at 100 they are.  Neither
    takes the form measured for the other; a third of the second's class does."""
    mk = lambda r: gpu.Solver(two_material_2d(n=n, kn_right=0.05, ratio=r, particles=200_000),
                              tally_faces=gpu.FACES_EVERY, T_init=seeded_temperature(n * n))
    a = mk(first)
    _settle(a)
    b = mk(second)
    assert b.march_tuning()[0] is None
    _settle(b)
    for s, r in ((a, first), (b, second)):
        measured = {k for k, v in s.march_tuning()[1].items() if v is not None}
        assert ("blocks" in measured) == (r == 100.0)
        assert s.step(1) == 0 and s.march_form() == s.march_tuning()[0]
    assert mk(second).march_tuning()[0] == b.march_tuning()[0]


def test_row_stripes_are_timed_beside_blocks(gpu):
    """Far flights on paths of many cells: both forms are candidates, and every
    iteration of the search gives the tiles' tallies."""
    w = two_material_2d(n=75, kn_right=0.6, ratio=12.0, particles=150_000)
    kw = dict(tally_faces=gpu.FACES_EVERY, T_init=seeded_temperature(w.n_cells))
    s, ref = gpu.Solver(w, **kw), gpu.Solver(w, march=1, **kw)
    ran = []
    for _ in range(6):
        assert s.step(1) == 0 and ref.step(1) == 0
        ran.append(s.march_form())
        ts, tr = s.tallies(), ref.tallies()
        for k in ts:
            assert torch.equal(ts[k], tr[k]), (ran, k)
    assert {"stripes", "blocks"} <= set(ran)
    assert {"stripes", "blocks"} <= {k for k, v in s.march_tuning()[1].items() if v is not None}


def test_forms_without_face_tallies(oracle_mod, gpu):
    """Short far flights: tiles and blocks are timed once most emitters fly, and
    each iteration gives the oracle's tallies in either."""
    w = two_material_2d(n=61, kn_right=0.05, ratio=30.0, particles=300_000)
    o, s = _pair(oracle_mod, gpu, w, tally_faces=oracle_mod.FACES_OFF,
                 T_init=seeded_temperature(w.n_cells))
    ran = []
    for i in range(9):
        assert o.step(1) == 0 and s.step(1) == 0
        ran.append(s.march_form())
        _same_cells(o, s, f"it{i} {ran}")
    assert ran[1:7] == ["tiles256", "blocks"] * 3 and ran[7] == ran[8]
    # from cold cells the search has not begun while only the walls emit
    c = gpu.Solver(two_material_2d(n=77, kn_right=0.02, ratio=30.0, particles=300_000),
                   tally_faces=gpu.FACES_OFF, T_init=np.full(77 * 77, 1.0))
    for _ in range(3):
        assert c.step(1) == 0
        if 2 * c.stats()["flights"] < c.stats()["n_emitters"] * c.stats()["n_per_emitter"]:
            assert c.march_form() == "tiles256"


@pytest.mark.parametrize("K,timed", [(2, False), (8, True)])
def test_forms_of_bands_without_face_tallies(gpu, K, timed):
    """Two bands on paths longer than the mesh keep to tiles, eight of which most
    are short time blocks as well; every iteration gives the tiles' tallies."""
    w = nongray_two_material_2d(n=64, K=K, ratio=20.0, particles=K * 16 * (64 * 64 + 256))
    kw = dict(tally_faces=gpu.FACES_OFF, T_init=seeded_temperature(64 * 64))
    s, ref = gpu.Solver(w, **kw), gpu.Solver(w, march=1, **kw)
    ran = []
    for _ in range(4):
        assert s.step(1) == 0 and ref.step(1) == 0
        ran.append(s.march_form())
        ts, tr = s.tallies(), ref.tallies()
        for k in ("D", "W", "B"):
            assert torch.equal(ts[k], tr[k]), (ran, k)
        assert torch.equal(s.state()[3], ref.state()[3])
    assert ("blocks" in ran) == timed
    assert ref.march_form() == "tiles256"


def test_bands_beyond_the_blocks_tables_keep_row_stripes(gpu):
    """Eighty bands of 560 x 560 cells are more blocks than a launch holds: the
    bands with long paths run by row stripes, as without blocks."""
    w = nongray_two_material_2d(n=560, K=80, particles=1)
    s = gpu.Solver(w, tally_faces=gpu.FACES_EVERY)
    ref = gpu.Solver(w, tally_faces=gpu.FACES_EVERY, march=1)
    assert s.step(1) == 0 and ref.step(1) == 0
    assert s.march_form() == "stripes" and ref.march_form() == "tiles256"
    ts, tr = s.tallies(), ref.tallies()
    for k in ts:
        assert torch.equal(ts[k], tr[k]), k


def _bands_2d(nx, ny, lam, ratio, per):
    """Bands of free paths lam (in cells; right half, ratio times that left)."""
    K = len(lam)
    w = nongray_two_material_2d(n=ny, K=K, particles=per * K * (nx * ny + 2 * (nx + ny)))
    w.nx, w.dx = nx, w.dy
    left = np.tile(np.arange(nx) < nx // 2, ny)
    w.tau = np.concatenate([np.where(left, v * ratio, v) * w.dx / g for v, g in zip(lam, w.band_vg)])
    w.wall_T = np.concatenate([np.full(2 * ny + nx, 0.99), np.full(nx, 1.01)])
    w.source = None
    return w


@pytest.mark.parametrize("nx,ny,lam,per,first,timed", [
    # (long paths, many rounds of few flights; long paths, few rounds)
    (376, 97, (2734.0, 242.0), 10, "stripes", {"tiles256", "blocks", "stripes"}),
    (96, 90, (700.0, 80.0), 20, "blocks", {"tiles256", "blocks", "stripes"}),
    (43, 215, (93.0, 40.0, 20.0, 10.0, 5.0, 2.0), 3, "tiles256", {"tiles256", "blocks"}),
    (60, 61, (90.0, 10.0), 60, "blocks", set()),
])
def test_form_of_bands_with_face_tallies(gpu, nx, ny, lam, per, first, timed):
    w = _bands_2d(nx, ny, lam, 20.0, per)
    kw = dict(tally_faces=gpu.FACES_EVERY, T_init=seeded_temperature(nx * ny))
    s, ref = gpu.Solver(w, **kw), gpu.Solver(w, march=1, **kw)
    ran = []
    for _ in range(2 + 3 * len(timed)):
        assert s.step(1) == 0 and ref.step(1) == 0
        ran.append(s.march_form())
        ts, tr = s.tallies(), ref.tallies()
        for k in ts:
            assert torch.equal(ts[k], tr[k]), (ran, k)
    assert ran[0] == first and set(ran[1:]) == (timed or {first})
    assert {k for k, v in s.march_tuning()[1].items() if v is not None} == timed


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_records_are_held_only_while_a_form_needs_them(gpu):
    """Two materials, 1e6 flights: 128 MB of block records, 84 MB of stripe records.
    None where no iteration runs by blocks; only the kept form's after a search."""
    def held(steps, n=140, **kw):
        w = two_material_2d(n=n, kn_right=kw.pop("kn"), ratio=30.0, particles=1_000_000)
        kw = dict(dict(T_init=seeded_temperature(w.n_cells)), **kw)
        before = _free()
        s = gpu.Solver(w, **kw)
        for _ in range(steps):
            assert s.step(1) == 0
        mb = (before - _free()) / 2 ** 20
        form = s.march_form()
        s.close()
        return mb, form

    held(1, kn=0.3, tally_faces=gpu.FACES_EVERY)                        # (first launches)
    mb, form = held(1, kn=0.3, tally_faces=gpu.FACES_OFF)               # paths of 42 cells: tiles
    assert form == "tiles256" and mb < 40
    mb, _ = held(1, kn=0.3, tally_faces=gpu.FACES_EVERY, n=141)         # searching
    assert mb > 190
    mb, form = held(6, kn=0.3, tally_faces=gpu.FACES_EVERY, n=142)      # settled
    assert mb < {"blocks": 170, "stripes": 125, "tiles512": 40}[form]
    mb, again = held(1, kn=0.3, tally_faces=gpu.FACES_EVERY, n=142)     # known from the start
    assert again == form and mb < {"blocks": 170, "stripes": 125, "tiles512": 40}[form]


@pytest.mark.parametrize("name", list(BLOCKS))
@pytest.mark.parametrize("faces", [True, False])
def test_blocks_run_where_they_are_meant_to(oracle_mod, gpu, name, faces):
    """The domain-block cases again, over enough iterations that blocks run twice
    (rays: in every one), on states that blocks have made as well."""
    make, kw = BLOCKS[name]
    w = make()
    kw = dict({"T_init": seeded_temperature(w.n_cells)}, **kw)
    if isinstance(kw["T_init"], str):       # (only the walls emit at first)
        kw["T_init"] = np.full(w.n_cells, w.t_ref)
    mode = oracle_mod.FACES_EVERY if faces else oracle_mod.FACES_OFF
    o, s = _pair(oracle_mod, gpu, w, tally_faces=mode, **kw)
    ran = []
    for i in range(5):
        assert o.step(1) == 0 and s.step(1) == 0
        ran.append(s.march_form())
        (_same_iteration if faces else _same_cells)(o, s, f"{name} it{i} {ran}")
    if "estimator" in kw:
        assert ran == ["blocks"] * 5
    elif faces:
        assert ran.count("blocks") >= 2 or set(ran) >= {"stripes", "blocks"}, ran
    elif name in ("null_few_flights", "null_no_weight"):    # (paths of 14 cells, cold at first)
        assert ran[0] == "tiles256"
    else:
        assert ran.count("blocks") >= 1, ran
