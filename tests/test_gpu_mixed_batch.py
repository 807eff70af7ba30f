"""Batches with lattices at tau = 1 and off it: FP32 and FP64 step the two kinds with
kernels of their own, each leaving out the other's tiles.  Every lattice against its
own run alone, bit for bit, one step a pass and two, by graph replays and direct
launches, and from grids of fewer blocks than tiles (each block then takes several,
of one kind and the other)."""
import numpy as np
import pytest

from gpu_common import gpu_lattice, need_gpu
from paper_1004_5058_amd import inputs

pytestmark = pytest.mark.gpu
STEPS = 26


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _specs(taus):
    """Uneven lattices with and without walls, their tau's in turn."""
    specs = []
    for k, (nx, ny, walls) in enumerate([(200, 72, True), (301, 41, False), (130, 97, True), (61, 9, False),
                                         (7, 33, True), (512, 24, True)]):
        ra, rb = inputs.emulsion(nx, ny, seed=60 + k)
        u = 0.01 * (1 + k % 3) if walls else 0.0
        specs.append(dict(nx=nx, ny=ny, rho_a=ra, rho_b=rb, ux=None, uy=None, walls=walls, u_top=u, u_bot=-u,
                          g_aa2=7.9 + 0.05 * k, tau=taus[k % len(taus)], fx_amp=2e-5, fx_k=0.3))
    return specs


_ALONE = {}


def _alone(storage, taus):
    """Fields, stress and profile of every lattice run alone, one step a pass."""
    if (storage, taus) not in _ALONE:
        out = []
        for s in _specs(taus):
            nx, ny, ra, rb, ux, uy = (s.pop(q) for q in ("nx", "ny", "rho_a", "rho_b", "ux", "uy"))
            lat = gpu_lattice(nx, ny, ra, rb, ux, uy, storage=storage, profile=True, **s)
            lat.step(STEPS)
            out.append((lat.fields(), lat.stress(), lat.profile()[0]))
            lat.close()
        _ALONE[storage, taus] = out
    return _ALONE[storage, taus]


def _check(b, storage, taus):
    sb, st, n = b.stress()
    assert n == STEPS
    for k, (fields, stress, prof) in enumerate(_alone(storage, taus)):
        for x, y in zip(b.fields(k), fields):
            np.testing.assert_array_equal(x, y, err_msg=f"lattice {k}")
        assert (sb[k], st[k], n) == stress, k
        # (its sums are grouped by tiles)
        assert np.max(np.abs(b.profile(k)[0] - prof)) <= 1e-13 * np.max(np.abs(prof)), k


@pytest.mark.parametrize("graph", [0, 6])
@pytest.mark.parametrize("storage,lanes", [("f32", 0), ("f32", 128), ("f32", 192), ("f32", 256), ("f64", 0), ("f16dev", 0),
                                           ("f16dev", 128), ("bf16dev", 256)])
def test_mixed_batch_equals_each_lattice_alone(storage, lanes, graph):
    from paper_1004_5058_amd import lb
    taus = (1.0, 1.2)
    b = lb.Batch(_specs(taus), storage=storage, profile=True)
    b.set_graph(graph)
    if lanes:
        b.set_fusion_tile(lanes)
        b.set_fusion(2, 12)
        assert b.launch()["steps_per_pass"] == 2
    b.step(12)
    b.step(STEPS - 12)
    _check(b, storage, taus)
    b.close()


@pytest.mark.parametrize("storage,per_pass", [("f32", 1), ("f32", 2), ("f64", 1)])
def test_every_replay_matches_direct_launches(storage, per_pass):
    """Graphs of such a batch have a branch for either kind: every replay against direct
    launches, with reads and a stress reset between the replays."""
    from paper_1004_5058_amd import lb
    graphed, direct = (lb.Batch(_specs((1.2, 1.0)), storage=storage, profile=True) for _ in range(2))
    for b, graph in ((graphed, 6), (direct, 0)):
        b.set_graph(graph)
        b.set_fusion(per_pass, 12 if per_pass == 2 else 0)
    for k in range(6):
        for b in (graphed, direct):
            b.step(6 if k % 2 else 13)
        for q in range(graphed.n):
            for x, y in zip(graphed.fields(q), direct.fields(q)):
                np.testing.assert_array_equal(x, y, err_msg=f"replay {k}, lattice {q}")
            np.testing.assert_array_equal(graphed.profile(q)[0], direct.profile(q)[0])
        for x, y in zip(graphed.stress(), direct.stress()):
            np.testing.assert_array_equal(x, y)
        if k == 2:
            for b in (graphed, direct):
                b.stress_reset()
    graphed.close()
    direct.close()


@pytest.mark.parametrize("n,nx,ny,per_pass", [(20, 256, 128, 1), (20, 256, 128, 2), (6, 128, 64, 1)])
def test_mixed_batch_takes_little_longer_than_either_kind(n, nx, ny, per_pass):
    """A step of the batch takes less than 1.5 times that of the slower kind alone (each
    kernel over all tiles, one after the other: 1.4 to 3.3 times)."""
    from paper_1004_5058_amd import lb
    ra, rb = inputs.noise(nx, ny, 1)
    times = []
    for taus in ((1.0,), (1.2,), (1.0, 1.2)):
        b = lb.Batch([dict(nx=nx, ny=ny, rho_a=ra, rho_b=rb, ux=None, uy=None, tau=taus[k % len(taus)]) for k in range(n)],
                     storage="f32", profile=False)
        b.set_fusion(per_pass)
        b.time_steps(512)
        times.append(min(b.time_steps(128) for _ in range(8)))
        b.close()
    assert times[2] <= 1.5 * max(times[:2]), times


SHAPES = [("f32", 64, 5), ("f32", 128, 11), ("f32", 512, 16), ("f64", 64, 7), ("f64", 256, 9), ("mom32", 64, 6),
          ("mom32", 256, 13)]


@pytest.mark.parametrize("grid", [1, 3, 8, 13])
@pytest.mark.parametrize("storage,bx,ly,taus", [(*s, (1.0,)) for s in SHAPES] + [(*s, (1.2, 1.0)) for s in SHAPES[:5]])
def test_fewer_blocks_than_tiles(storage, bx, ly, grid, taus):
    from paper_1004_5058_amd import lb
    b = lb.Batch(_specs(taus), storage=storage, profile=True)
    b.set_launch(bx, ly, grid)
    assert b.launch()["grid"] == grid
    b.step(STEPS)
    _check(b, storage, taus)
    b.close()
