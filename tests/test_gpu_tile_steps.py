"""Launches that advance two or three time steps of a lattice that does not fill
the chip (FP32 storage, one row per wavefront): the same bits as one step per
launch, for every boundary kind, with and without the Navier-Stokes correction.
Calls of one step always take the single-step launches, so they are the
reference."""
import numpy as np
import pytest

from paper_1903_01168_amd import capi
from paper_1903_01168_amd import workloads as W

pytestmark = pytest.mark.gpu


def _lattice(nx, ny, bc_x, bc_y, nsc):
    p = W.params(nx=nx, ny=ny, bc_x=bc_x, bc_y=bc_y, rho0_r=2.0, rho0_b=1.0, tau_r=0.8, tau_b=0.9, A=1e-3,
                 storage="f32", collision="mrt" if nsc or nx % 2 else "bgk", ns_correction=nsc,
                 gx=1e-5 if bc_y == "walls" else 0.0,
                 u_in_r=0.01, u_in_b=0.01, p_out=0.48, contact_angle=60.0 if bc_y == "walls" else -1.0)
    g = capi.Lattice(p)
    rng = np.random.default_rng(nx + ny)
    f = np.clip(1.5 * np.sin(np.arange(nx) * 0.37)[None, :] * np.cos(np.arange(ny) * 0.23)[:, None] + 0.5
                + 0.1 * rng.random((ny, nx)), 0.0, 1.0)
    g.init(2.0 * f, 1.0 - f, 0.02 * (rng.random((ny, nx)) - 0.5), 0.02 * (rng.random((ny, nx)) - 0.5))
    if bc_x == "open":
        g.set_inlet_color(np.where(np.arange(ny) % 3 > 0, 1, -1).astype(np.int8))
    return g


# around the 54 (48 between walls) columns and 2 or 6 rows of a workgroup of three steps, narrower and flatter than
# it, and the largest of one round of workgroups; two steps in one round and in two; just beyond
SHAPES = [(64, 64), (54, 6), (55, 7), (47, 95), (49, 13), (7, 5), (2, 30), (97, 4), (33, 5), (300, 200), (2592, 25),
          (319, 321), (59, 1201), (512, 512), (647, 290), (541, 520)]


@pytest.mark.parametrize("nsc", [False, True])
@pytest.mark.parametrize("bc_y", ["periodic", "walls", "freeslip", "slip_top"])
@pytest.mark.parametrize("bc_x", ["periodic", "open"])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_tile_steps_bit_identical(nx, ny, bc_x, bc_y, nsc):
    with _lattice(nx, ny, bc_x, bc_y, nsc) as a, _lattice(nx, ny, bc_x, bc_y, nsc) as b:
        a.step(7)
        for _ in range(7):
            b.step(1)
        assert np.isfinite(b.get_pops()).all()
        assert a.get_pops().tobytes() == b.get_pops().tobytes()


def test_any_number_of_steps_bit_identical():
    """Launches of three steps, single steps for the rest, and graph replays of either parity."""
    with _lattice(100, 100, "periodic", "walls", True) as a, _lattice(100, 100, "periodic", "walls", True) as b:
        a.step(167)
        for n in (1, 2, 3, 5, 7, 61, 73, 15):
            b.step(n)
        assert a.steps_done == b.steps_done == 167
        assert a.get_pops().tobytes() == b.get_pops().tobytes()


@pytest.mark.parametrize("n,nsc", [(3, False), (5, True), (9, False)])
def test_batch_tile_steps_bit_identical(n, nsc):
    """Batches of small lattices, two groups in flight: pairs of two-step launches, single steps for the rest."""
    kinds = [("periodic", "periodic"), ("open", "freeslip"), ("periodic", "walls"), ("open", "slip_top")]
    args = [(61 + 23 * k, 40 + 17 * k) + kinds[k % 4] + (nsc,) for k in range(n)]
    alone, mixed = [_lattice(*a) for a in args], [_lattice(*a) for a in args]
    mixed[0].step(1)
    alone[0].step(1)
    b = capi.Batch(mixed)
    b.step(75)
    b.step(2)
    for g in alone:
        for _ in range(77):
            g.step(1)
    for g, m in zip(alone, mixed):
        assert g.get_pops().tobytes() == m.get_pops().tobytes()
    b.close()
    for g in alone + mixed:
        g.close()
