"""The multigrid CG's group beside other work: whichever workgroups the solve's
group is elected from, and however many of them, its result is the same bit for
bit (its values do not depend on the group)."""
import threading

import pytest

from synth import cavity_2d, seeded_temperature, two_material_2d

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_09465_amd as P
    P.library()
    return P


@pytest.mark.parametrize("n,waves", [(64, 0), (160, 0), (257, 0), (160, 4)])
def test_mg_solves_beside_long_particle_steps(gpu, n, waves):
    """Newton steps of three solvers from three threads, while particle steps that
    hold every compute unit for milliseconds run on a fourth stream."""
    w = cavity_2d(n=n, kn=0.1, particles=20 * n * n, newton=True)
    kw = dict(tally_faces=gpu.FACES_OFF, cg_precond=gpu.PRECOND_MG, own_stream=True, cg_waves=waves)
    alone = gpu.Solver(w, **kw)
    for _ in range(4):
        assert alone.step(1) == 0
    busy = gpu.Solver(two_material_2d(n=256, kn_right=0.05, ratio=50.0, particles=4_000_000), march=1,
                      tally_faces=gpu.FACES_EVERY, own_stream=True, T_init=seeded_temperature(256 * 256))
    ss = [gpu.Solver(w, **kw) for _ in range(3)]
    rcs = [None] * 4

    def work(i):
        rcs[i] = [(busy if i == 3 else ss[i]).step(1) for _ in range(4)]

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert rcs == [[0, 0, 0, 0]] * 4
    for s in ss:
        assert torch.equal(s.state()[2], alone.state()[2])
        assert s.stats()["cg_iters_total"] == alone.stats()["cg_iters_total"]
