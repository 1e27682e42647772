"""Grids of more than 2048 rows of cells: the one-kernel solve's forms for
them, and beyond 4096 rows, where the reduced systems of the PCR strategy are
solved in a kernel of their own."""
import numpy as np
import pytest

from paper_1611_05984_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _domain(nx, ny, maker, sponge, **params):
    from paper_1611_05984_amd import wavestep as ws
    dx = 0.05
    X = np.arange(nx + 1)[None, :] / nx
    Y = np.arange(ny + 1)[:, None] / ny
    z = -0.5 + 0.1 * np.sin(7 * X + 5 * Y + nx + ny)
    z = np.where((X > 0.6) & (Y > 0.6), z + 0.45, z)      # a bank that dries in places
    d = ws.Domain(nx, ny, dx, dx, wl.courant_dt(0.2, dx, 0.6), z, **params)
    if maker is not None:
        d.set_boundary(maker, ws.WAVES, 2, [0.02, 0.01], [1.5, 0.9], [0.3, -0.2], [0.0, 1.0])
    if sponge is not None:
        d.set_boundary(sponge, ws.SPONGE, 5)
    d.apply_edit(ws.EDIT_WATER, 0.4 * nx * dx, 0.4 * ny * dx, 0.03, 6 * dx)
    return d


def _near(a, b):
    """The bound the solve strategies are held to among each other."""
    for x, y in zip(a.state_numpy(), b.state_numpy()):
        assert np.isfinite(x).all() and np.abs(x - y).max() <= 1e-6 * max(1.0, np.abs(x).max())


def _equal(a, b):
    for x, y in zip(a.state_numpy(), b.state_numpy()):
        assert np.isfinite(x).all() and np.array_equal(x, y)


# up to 512 columns rows and columns share a launch (4 columns a workgroup), beyond that
# the rows have one of their own; a batch always shares it, at 8 columns
@pytest.mark.parametrize("nx,ny,maker,sponge", [
    (3, 2049, 3, 1), (511, 2081, 2, 0), (512, 4096, 0, 3), (513, 2049, 1, 2), (1001, 4095, 2, 1),
])
def test_tall_forms(nx, ny, maker, sponge):
    from paper_1611_05984_amd import wavestep as ws
    print("case: tall %dx%d maker %s sponge %s" % (nx, ny, maker, sponge), flush=True)
    g, t, b, small = (_domain(nx, ny, maker, sponge), _domain(nx, ny, maker, sponge), _domain(nx, ny, maker, sponge),
                      _domain(50, 40, 0, 1))
    t.set_tuning(16, 128, ws.SOLVE_THOMAS)
    B = ws.Batch(2)
    B.attach(b)
    B.attach(small)
    for n in (1, 4):
        g.advance(n)
        t.advance(n)
        B.advance(n)
        B.sync()
        _near(g, t)
        _equal(g, b)
    B.close()


# reduced systems of 514, 1126 and 2048 unknowns: both register counts of every thread count
@pytest.mark.parametrize("nx,ny,maker,sponge", [(20, 4100, 0, 3), (70, 9000, 3, 1), (20, 16384, 2, 0)])
def test_pcr_beyond_4096_rows(nx, ny, maker, sponge):
    """The PCR kernel of the grids past the one-kernel solve: the same bits at
    every thread count, alone and in a batch beside a domain on the
    one-kernel path, and the Thomas path's result."""
    from paper_1611_05984_amd import wavestep as ws
    print("case: pcr %dx%d maker %s sponge %s" % (nx, ny, maker, sponge), flush=True)
    t = _domain(nx, ny, maker, sponge)
    t.set_tuning(16, 128, ws.SOLVE_THOMAS)
    t.advance(5)
    alone = []
    for threads in (64, 128, 256):
        d = _domain(nx, ny, maker, sponge)
        d.set_tuning(16, threads, ws.SOLVE_PCR)
        d.advance(5)
        alone.append(d)
    _near(alone[0], t)
    _equal(alone[0], alone[1])
    _equal(alone[0], alone[2])
    small = _domain(130, 90, 0, 1)
    small.advance(5)
    for threads in (64, 128, 256):
        b, s = _domain(nx, ny, maker, sponge), _domain(130, 90, 0, 1)
        B = ws.Batch(2)
        B.set_tuning(16, threads, ws.SOLVE_PCR)
        B.attach(b)
        B.attach(s)
        B.advance(5)
        B.sync()
        _equal(alone[0], b)
        _equal(small, s)
        B.close()
