"""The one-kernel solve of a pass at the edges of its segments, workgroups and
range, against the FP64 oracle: lines of one cell more and less than whole
16-cell segments, rows and columns of one segment, the longest columns it
takes with 16-cell segments (2048 cells) and the first with 32, a wave maker
and a sponge on each pair of sides.  The bounds are the parity tests'
for these step counts: 2e-6 of the wave height after one Euler step, 1e-5
after the first full step (times sqrt(g d) for the discharges)."""
import math

import numpy as np
import pytest

import oracle as o
from paper_1611_05984_amd import workloads as wl

pytestmark = pytest.mark.gpu
A0, DEPTH = 0.03, 0.5


def _pair(nx, ny, maker, sponge, **params):
    from paper_1611_05984_amd import wavestep as ws
    dx = 0.05
    rng = np.random.default_rng(nx * 7919 + ny)
    X = np.arange(nx + 1)[None, :] / nx
    Y = np.arange(ny + 1)[:, None] / ny
    z = -0.5 + 0.1 * np.sin(7 * X + 5 * Y + rng.uniform(0, 6)) * np.ones((ny + 1, nx + 1))
    z = np.where((X > 0.6) & (Y > 0.6), z + 0.45, z)      # a bank that dries in places
    z = z.astype(np.float32).astype(np.float64)
    dt = wl.courant_dt(0.2, dx, 0.6)
    g = ws.Domain(nx, ny, dx, dx, dt, z, **params)
    r = o.Domain(nx, ny, dx, dx, dt, z, **params)
    for d in (g, r):
        if maker is not None:
            d.set_boundary(maker, ws.WAVES, 2, [0.02, 0.01], [1.5, 0.9], [0.3, -0.2], [0.0, 1.0])
        if sponge is not None:
            d.set_boundary(sponge, ws.SPONGE, 5)
        d.apply_edit(ws.EDIT_WATER, 0.4 * nx * dx, 0.4 * ny * dx, A0, 6 * dx)
    return g, r


@pytest.mark.parametrize("nx,ny,maker,sponge", [
    (16, 16, 0, 1), (17, 15, 1, 2), (15, 17, 2, 0), (33, 2, 3, 0), (2, 31, None, 3), (129, 256, 0, 3),
    (130, 257, 3, 1), (1025, 48, 1, 3), (61, 512, 2, 1), (70, 1023, 3, 0), (9, 2048, 2, 1), (65, 2049, 0, 2),
])
def test_one_kernel_solve_edges(nx, ny, maker, sponge):
    print("case: solve %dx%d maker %s sponge %s" % (nx, ny, maker, sponge), flush=True)
    g, r = _pair(nx, ny, maker, sponge)
    for n, rel in ((1, 2e-6), (2, 1e-5)):
        g.advance(n)
        r.advance(n)
        got, want = g.state_numpy(), r.state()
        for k, (a, b) in enumerate(zip(got, want)):
            scale = A0 * (math.sqrt(9.81 * DEPTH) if k else 1.0)
            assert np.abs(a - b).max() <= rel * scale, (n, k, np.abs(a - b).max())
    assert g.query()[2] == 0


@pytest.mark.parametrize("nx,ny,maker,sponge", [(24, 4095, 3, 1), (17, 4096, 2, 0), (9, 2080, 3, 1), (130, 2050, 0, 3)])
def test_tall_columns_equal_thomas(nx, ny, maker, sponge):
    """Columns of more than 2048 cells (32-cell segments, rows in a launch of
    their own) against the lane-per-system Thomas path, within the bound the
    other strategies are held to; a batch with a small domain gives the same
    bits as alone."""
    from paper_1611_05984_amd import wavestep as ws
    print("case: tall %dx%d maker %s sponge %s" % (nx, ny, maker, sponge), flush=True)
    g, _ = _pair(nx, ny, maker, sponge)
    t, _ = _pair(nx, ny, maker, sponge)
    b, _ = _pair(nx, ny, maker, sponge)
    small, _ = _pair(40, 30, 0, 1)
    t.set_tuning(16, 128, ws.SOLVE_THOMAS)
    B = ws.Batch(2)
    B.attach(b)
    B.attach(small)
    for n in (1, 4):
        g.advance(n)
        t.advance(n)
        B.advance(n)
        B.sync()
        for x, y, z in zip(g.state_numpy(), t.state_numpy(), b.state_numpy()):
            assert np.abs(x - y).max() <= 1e-6 * max(1.0, np.abs(x).max())
            assert np.array_equal(x, z)
    B.close()


@pytest.mark.parametrize("solver", [1, 2])
def test_switching_solvers_keeps_the_one_kernel_path_right(solver):
    """Other strategies use the same scratch: PCR, the other, PCR again from
    one snapshot gives PCR's bits; likewise after a rejected terrain edit
    (which uses the cell-depth field) and after a boundary change."""
    from paper_1611_05984_amd import wavestep as ws
    g, _ = _pair(90, 50, 0, 3)
    g.advance(4)
    snap = g.snapshot()
    g.advance(5)
    want = g.state_numpy()
    g.set_tuning(8, 128, solver)
    g.restore(snap)
    g.advance(5)
    g.set_tuning(8, 128, ws.SOLVE_PCR)
    g.restore(snap)
    assert g.apply_edit(ws.EDIT_TERRAIN, 2.0, 1.0, -400.0, 0.05) == ws.ENOTDD
    g.advance(5)
    for a, b in zip(want, g.state_numpy()):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("nx,ny,sponge", [(62, 9, 1), (63, 40, 2), (130, 77, 3)])
def test_nlsw_passes_follow_model_changes(nx, ny, sponge):
    """NLSW passes write the discharges from the stencil and, alone, leave out
    the F*, G* history they know to be zero; a batch never leaves it out.  One
    start-up, then NLSW, the dispersive model and NLSW again: the same bits
    alone and in a batch, and the oracle's state within the parity bound."""
    from paper_1611_05984_amd import wavestep as ws
    print("case: nlsw %dx%d sponge %s" % (nx, ny, sponge), flush=True)
    a, r = _pair(nx, ny, 0, sponge, model=1)
    b, _ = _pair(nx, ny, 0, sponge, model=1)
    B = ws.Batch(1)
    slot = B.attach(b)
    for model, n in ((1, 5), (0, 4), (1, 2), (0, 3), (1, 6)):
        a.update(model=model)
        b.update(model=model)
        a.advance(n)
        B.advance(n)
        B.sync()
        for x, y in zip(a.state_numpy(), b.state_numpy()):
            assert np.isfinite(x).all() and np.array_equal(x, y), (model, n)
        if (model, n) == (1, 5):
            r.advance(5)
            for k, (x, y) in enumerate(zip(a.state_numpy(), r.state())):
                assert np.abs(x - y).max() <= 1e-5 * A0 * (math.sqrt(9.81 * DEPTH) if k else 1.0), k
    B.detach(slot)
    B.close()


@pytest.mark.parametrize("nx,ny,model", [(2, 2, 0), (17, 90, 0), (510, 3, 0), (300, 130, 1)])
def test_wave_makers_in_one_call_and_in_many(nx, ny, model):
    """A call of several steps evaluates the makers once a time level (in the
    predictor's launch), a call of one step both levels, a batch both in a
    launch of its own: the same bits, also where a call of each kind follows
    the other and where a second domain of the batch has no maker."""
    print("case: makers %dx%d model %d" % (nx, ny, model), flush=True)
    from paper_1611_05984_amd import wavestep as ws

    def make():
        d = _pair(nx, ny, 0, None, model=model)[0]
        d.set_boundary(ws.NORTH, ws.WAVES, 2, [0.01] * 3, [1.2, 0.8, 0.5], [1.7, 1.2, -0.4], [0.5, 2.0, 0.1])
        return d
    one, many, b = make(), make(), make()
    B = ws.Batch(2)
    still, _ = _pair(20, 20, None, 1, model=model)
    B.attach(still)
    slot = B.attach(b)
    for n in (7, 4):
        one.advance(n)
        for _ in range(n):
            many.advance(1)
        B.advance(n)
        B.sync()
        for x, y, z in zip(one.state_numpy(), many.state_numpy(), b.state_numpy()):
            assert np.isfinite(x).all() and np.array_equal(x, y) and np.array_equal(x, z), n
        B.detach(slot)
        b.advance(3)
        one.advance(3)
        many.advance(2)
        many.advance(1)
        slot = B.attach(b)
    B.close()
