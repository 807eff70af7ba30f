"""Lattices that run different step kernels (FP32 and FP64 at tau = 1 and off it, a
batch of both) have tuning-cache entries of their own; those of one kind share theirs."""
import json

import pytest

from gpu_common import gpu_lattice, need_gpu
from paper_1004_5058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f64", "bf16dev"])
def test_entries_per_kernel(tmp_path, storage):
    need_gpu()
    cache = str(tmp_path / "tune.json")
    ra, rb = inputs.noise(128, 64, 2)
    keys = []
    for tau in (1.0, 1.2, 0.9, 1.0):
        lat = gpu_lattice(128, 64, ra, rb, storage=storage, tau=tau)
        lat.autotune(cache, steps=2)
        lat.close()
        keys.append(set(json.load(open(cache))))
    own = storage != "bf16dev"
    assert len(keys[0]) == 1 and len(keys[1]) == (2 if own else 1)
    assert keys[2] == keys[1] == keys[3]


def test_batches_of_one_kind_and_of_both(tmp_path):
    need_gpu()
    from paper_1004_5058_amd import lb
    cache = str(tmp_path / "tune.json")
    ra, rb = inputs.noise(128, 64, 2)
    for taus, n in (((1.0, 1.0), 1), ((1.0, 1.2), 2), ((0.9, 1.2), 3), ((1.3, 1.0), 3)):
        b = lb.Batch([dict(nx=128, ny=64, rho_a=ra, rho_b=rb, ux=None, uy=None, tau=t) for t in taus], storage="f32",
                     profile=False)
        b.autotune(cache, steps=2)
        b.close()
        assert len(json.load(open(cache))) == n
