"""The tau = 1 step kernels at the edges of their tiles: one column and row more
or less than a wave's 60 (58 in the moment form) output columns, a 128, 192, 256
or 512 column tile and a fused tile's 118 / 182 / 246; lattices lower than the
five rows of the force stencil; segments that end on a partial group of eight
profile rows.  Fields against the FP64 oracle after 12 steps and the accumulated
line profile against the mean of the oracle's, to the bounds of the randomized
sweep: FP64 and FP64 moments 1e-12, FP32 and FP32 moments 1e-6, FP16 5e-4 (the
same noise start, fewer steps)."""
import struct

import numpy as np
import pytest

from gpu_common import compare_fields, gpu_lattice, need_gpu, oracle_params
from oracle import oracle as O
from paper_1004_5058_amd import inputs

pytestmark = pytest.mark.gpu
HEADER = 72                      # bytes; its last three 64-bit words are the section sizes
TOL = {"f64": 1e-12, "f32": 1e-6, "f16dev": 5e-4, "mom64": 1e-12, "mom32": 1e-6}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


_ORACLE = {}


def _oracle(nx, ny, walls):
    """Oracle start densities, state after 12 steps and mean line profile of the 12."""
    key = (nx, ny, walls)
    if key not in _ORACLE:
        ra, rb = inputs.noise(nx, ny, 3)
        u = 0.01 if walls else 0.0
        p = oracle_params(nx, ny, walls, u, -u)
        f = O.init(p, ra, rb, None, None)
        mean = np.zeros(ny)
        for _ in range(12):
            mean += O.fields(p, f)[2].mean(axis=1) / 12
            f = O.run(p, f, 1)[0]
        _ORACLE[key] = ra, rb, u, p, f, mean
    return _ORACLE[key]


CASES = [("f64", bx, 0) for bx in (64, 128, 256)] + [("f32", bx, 0) for bx in (64, 256, 512)] + \
        [("f32", 64, lanes) for lanes in (128, 192, 256)] + [("f16dev", bx, 0) for bx in (64, 512)] + \
        [("f16dev", 64, lanes) for lanes in (128, 192, 256)] + [("mom64", 64, 0), ("mom32", 64, 0), ("mom32", 256, 0)]


@pytest.mark.parametrize("storage,bx,lanes", CASES)
@pytest.mark.parametrize("nx,ny,walls", [(1, 2, False), (58, 3, True), (60, 4, True), (61, 5, False), (119, 11, True),
                                         (183, 17, False), (257, 9, True), (513, 26, True)])
def test_tile_edges_match_oracle(storage, bx, lanes, nx, ny, walls):
    ra, rb, u, p, g, mean = _oracle(nx, ny, walls)
    profile = storage != "f16dev"         # (with a profile FP16 runs the general kernels)
    lat = gpu_lattice(nx, ny, ra, rb, walls=walls, u_top=u, u_bot=-u, storage=storage, profile=profile)
    lat.set_launch(bx, 11)
    if lanes:
        lat.set_fusion_tile(lanes)
        lat.set_fusion(2, 11)
    lat.step(12)
    tol = TOL[storage]
    compare_fields(lat, p, g, tol)
    if profile:
        prof, n = lat.profile()
        assert n == 12
        assert np.max(np.abs(prof - mean)) <= tol
    lat.close()


@pytest.mark.parametrize("storage,width", [("f64", 64), ("mom32", 60)])
def test_checkpoint_with_fewer_profile_rows(storage, width):
    """A checkpoint whose profile has a row per `width` columns, as these forms
    kept it before, fills the first of the rows kept now; their sums are read."""
    nx, ny = 130, 9
    ra, rb, u, *_ = _oracle(nx, ny, True)
    kw = dict(walls=True, u_top=u, u_bot=-u, storage=storage, profile=True)
    lat = gpu_lattice(nx, ny, ra, rb, **kw)
    lat.step(6)
    buf = lat.save()
    want = lat.profile()[0]
    fb, sb, pb = struct.unpack_from("<QQQ", buf.tobytes(), HEADER - 24)
    rows = buf[HEADER + fb + sb:].view(np.float64).reshape(-1, ny)
    fewer = np.zeros((-(-nx // width), ny))
    fewer[1] = rows.sum(axis=0)
    old = np.concatenate([buf[:HEADER - 8], np.array([fewer.nbytes], np.uint64).view(np.uint8),
                          buf[HEADER:HEADER + fb + sb], fewer.reshape(-1).view(np.uint8)])
    other = gpu_lattice(nx, ny, ra, rb, **kw)
    other.step(2)
    other.load(old)
    np.testing.assert_allclose(other.profile()[0], want, rtol=1e-14, atol=0)
    other.close()
    lat.close()


@pytest.mark.parametrize("storage,tau", [("f32", 1.0), ("f16dev", 1.0), ("f32", 1.2), ("bf16dev", 1.0)])
def test_pairs_left_to_choose_equal_set_tiles(storage, tau):
    """Two steps a pass of a small lattice: the library's own choice (single steps)
    against a set tile (the fused kernel), across graph replays and an odd remainder."""
    ra, rb, u, *_ = _oracle(183, 17, False)
    pops = []
    for ly2 in (0, 6):
        lat = gpu_lattice(183, 17, ra, rb, walls=False, storage=storage, tau=tau)
        lat.set_graph(6)
        lat.set_fusion(2, ly2)
        assert lat.launch()["steps_per_pass"] == 2
        lat.step(8)
        lat.step(15)
        assert lat.time() == 23
        pops.append(lat.populations())
        lat.close()
    np.testing.assert_array_equal(pops[0], pops[1])
