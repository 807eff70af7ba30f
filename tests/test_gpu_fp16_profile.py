"""An FP16 lattice evolves the same whether or not its line profile is
accumulated: one rule defines the stored values of every kernel, so populations
and wall stresses are equal to the bit with the profile on and off, one step a
pass and two (set tiles: the fused kernel runs), alone and in a batch."""
import numpy as np
import pytest

from gpu_common import gpu_lattice, need_gpu
from paper_1004_5058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("nx,ny,walls", [(183, 37, True), (130, 21, False)])
@pytest.mark.parametrize("lanes", [0, 128, 256])
def test_profile_does_not_change_the_run(nx, ny, walls, lanes):
    ra, rb = inputs.emulsion(nx, ny, seed=4)
    u = 0.02 if walls else 0.0
    runs = []
    for profile in (False, True):
        lat = gpu_lattice(nx, ny, ra, rb, walls=walls, u_top=u, u_bot=-u, storage="f16dev", profile=profile,
                          fx_amp=2e-5, fx_k=0.3)
        if lanes:
            lat.set_fusion_tile(lanes)
            lat.set_fusion(2, 12)
        lat.step(25)
        runs.append((lat.populations(), lat.stress()))
        lat.close()
    np.testing.assert_array_equal(runs[1][0], runs[0][0])
    assert runs[1][1] == runs[0][1]


@pytest.mark.parametrize("per_pass", [1, 2])
def test_batch_equals_single_lattice_without_profile(per_pass):
    from paper_1004_5058_amd import lb
    specs = []
    for k, (nx, ny) in enumerate([(128, 64), (75, 33)]):
        ra, rb = inputs.emulsion(nx, ny, seed=9 + k)
        specs.append(dict(nx=nx, ny=ny, rho_a=ra, rho_b=rb, ux=None, uy=None, u_top=0.01, u_bot=-0.01))
    b = lb.Batch(specs, storage="f16dev", profile=True)
    b.set_fusion(per_pass, 12 if per_pass == 2 else 0)
    b.step(20)
    sb, st, n = b.stress()
    for k, s in enumerate(specs):
        lat = gpu_lattice(s["nx"], s["ny"], s["rho_a"], s["rho_b"], u_top=0.01, u_bot=-0.01, storage="f16dev")
        lat.step(20)
        for x, y in zip(b.fields(k), lat.fields()):
            np.testing.assert_array_equal(x, y)
        assert (sb[k], st[k], n) == lat.stress()
        lat.close()
    b.close()
