"""FP32 rest populations of 16-bit storage are rounded to a grid of two ulps (the
lowest bit is a flag), around powers of two, at zero and at tiny values too."""
import numpy as np
import pytest

from paper_1903_01168_amd import capi
from paper_1903_01168_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f16s", "bf16s"])
def test_rest_rounds_to_nearest_of_its_grid(storage):
    nx, ny = 64, 64
    p = W.params(nx=nx, ny=ny, bc_x="periodic", bc_y="periodic", rho0_r=2.0, rho0_b=1.0, storage=storage)
    rng = np.random.default_rng(5)
    v = np.float32(rng.random((2, ny, nx)) * 2.5)
    powers = np.float32(2.0) ** np.arange(-60, 3, dtype=np.float32)
    edge = np.stack([(powers.view(np.uint32) + np.uint32(k & 0xffffffff)).view(np.float32) for k in range(-4, 5)])
    v[:, :9, :63] = edge
    v[:, 10] = 0.0
    v[:, 11, ::2] *= -1e-6
    v[:, 12] = np.float32(1e-39)               # subnormal
    pops = np.zeros((2, 9, ny, nx))
    pops[:, 0] = v
    with capi.Lattice(p) as g:
        g.set_pops(pops)
        out = g.get_pops()[:, 0]
    # half a cell of two ulps, and the decoder's rounding of reference + deviation
    assert (np.abs(out - v) <= 1.5 * np.spacing(np.abs(v)).astype(float)).all()
    assert (out[:, 10] == 0.0).all()
