"""The steps per pass that lb_get_launch reports are those that run, also on
small states with everything else at its default: the two-step kernel keeps its
line-profile partial sums in rows of their own, behind the single-step kernel's
one per 64 columns, and a checkpoint holds them."""
import struct

import numpy as np
import pytest

from gpu_common import gpu_lattice, need_gpu
from paper_1004_5058_amd import inputs

pytestmark = pytest.mark.gpu
HEADER = 72                      # bytes; its last three 64-bit words are the section sizes


@pytest.mark.parametrize("storage,tau", [("f32", 1.0), ("f32", 1.2), ("f16dev", 1.0), ("bf16dev", 1.0)])
@pytest.mark.parametrize("nx,ny", [(130, 24), (300, 96)])
@pytest.mark.parametrize("graph", [0, 4])
def test_reported_steps_per_pass_run(storage, tau, nx, ny, graph):
    need_gpu()
    ra, rb = inputs.emulsion(nx, ny, seed=6)
    for per_pass in (1, 2):
        lat = gpu_lattice(nx, ny, ra, rb, u_top=0.02, u_bot=-0.02, storage=storage, profile=True, tau=tau)
        lat.set_graph(graph)
        lat.set_fusion(per_pass)
        assert lat.launch()["steps_per_pass"] == per_pass
        lat.step(8)
        buf = lat.save()
        lat.close()
        fb, sb, pb = struct.unpack_from("<QQQ", buf.tobytes(), HEADER - 24)
        rows = buf[HEADER + fb + sb:HEADER + fb + sb + pb].view(np.float64).reshape(-1, ny)
        single = -(-nx // 60) if storage == "f32" and tau == 1.0 else -(-nx // 64)    # rows the single steps fill
        assert np.any(rows[:single] != 0) == (per_pass == 1)
        assert np.any(rows[single:] != 0) == (per_pass == 2)
