"""Launches that advance two time steps (planned for lattices of 500 000 nodes
and more in FP32 storage wherever a call has at least four steps): the same bits
as one step per launch, for every boundary kind and ragged shape.  Calls of one
step always take the single-step launches, so they are the reference."""
import numpy as np
import pytest

from paper_1903_01168_amd import capi
from paper_1903_01168_amd import workloads as W

pytestmark = pytest.mark.gpu


def _params(nx, ny, bc_x, bc_y, collision="bgk"):
    return W.params(nx=nx, ny=ny, bc_x=bc_x, bc_y=bc_y, rho0_r=2.0, rho0_b=1.0, tau_r=0.8, tau_b=0.9, A=1e-3,
                    storage="f32", collision=collision, gx=1e-5 if bc_y == "walls" else 0.0, u_in_r=0.01, u_in_b=0.01,
                    p_out=0.48, contact_angle=60.0 if bc_y == "walls" else -1.0)


def _fields(nx, ny, seed):
    """Mixed and pure nodes, rough at the scale of a few nodes."""
    rng = np.random.default_rng(seed)
    f = np.clip(1.5 * np.sin(np.arange(nx) * 0.37 + rng.random() * 6)[None, :]
                * np.cos(np.arange(ny) * 0.23 + rng.random() * 6)[:, None] + 0.5 + 0.1 * rng.random((ny, nx)), 0.0, 1.0)
    return 2.0 * f, 1.0 - f, 0.02 * (rng.random((ny, nx)) - 0.5), 0.02 * (rng.random((ny, nx)) - 0.5)


def _lattice(p, seed=1):
    g = capi.Lattice(p)
    g.init(*_fields(p["nx"], p["ny"], seed))
    if p["bc_x"] == "open":
        g.set_inlet_color(np.where(np.arange(p["ny"]) % 3 > 0, 1, -1).astype(np.int8))
    return g


def _bits(g):
    """The stored populations of the lattice's own columns (a saved state also holds the padding of each row)."""
    return np.ascontiguousarray(g.get_pops()).tobytes()


def _same(p, steps, tx=0, strip=0):
    with _lattice(p) as a, _lattice(p) as b:
        a.set_launch(tx, strip)
        a.step(steps)
        for _ in range(steps):
            b.step(1)
        assert _bits(a) == _bits(b)


# widths around multiples of the 58 (54 next to walls) columns of a wavefront and of the 64-column blocks, one
# narrower than a wavefront, the narrowest and the flattest; strips of one row, of several and of the whole height
SHAPES = [(232, 2160, 0, 0), (1000, 517, 64, 5), (59, 8500, 128, 1), (17, 29500, 0, 64), (125003, 4, 256, 3),
          (541, 929, 256, 16)]


@pytest.mark.parametrize("bc_y", ["periodic", "walls", "freeslip", "slip_top"])
@pytest.mark.parametrize("bc_x", ["periodic", "open"])
@pytest.mark.parametrize("nx,ny,tx,strip", SHAPES)
def test_f32_two_steps_bit_identical(nx, ny, tx, strip, bc_x, bc_y):
    _same(_params(nx, ny, bc_x, bc_y, "mrt" if nx % 2 else "bgk"), 8, tx, strip)


def test_any_number_of_steps_bit_identical():
    """Pairs of two-step launches, single steps for the rest, and graph replays
    of either parity give the same bits however a run is cut into calls."""
    p = _params(1000, 517, "periodic", "walls")
    with _lattice(p) as a, _lattice(p) as b:
        a.step(167)
        for n in (1, 2, 3, 5, 7, 64, 70, 15):
            b.step(n)
        assert a.steps_done == b.steps_done == 167 and _bits(a) == _bits(b)


def test_batch_two_steps_bit_identical():
    """Two groups of a batch, in flight together, against single steps."""
    ps = [_params(700, 430, "periodic", "periodic"), _params(613, 410, "open", "freeslip"),
          _params(500, 333, "periodic", "walls")]
    alone, mixed = [_lattice(p, k) for k, p in enumerate(ps)], [_lattice(p, k) for k, p in enumerate(ps)]
    b = capi.Batch(mixed)
    b.step(75)
    b.step(2)
    for g in alone:
        for _ in range(77):
            g.step(1)
    for g, m in zip(alone, mixed):
        assert _bits(g) == _bits(m)
    b.close()
    for g in alone + mixed:
        g.close()
