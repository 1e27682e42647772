"""Calls between the steps of a running domain (autotuner, boundary and model
changes, terrain edits) against the same run without them or with the GPU
waited for in between: the same bits."""
import numpy as np
import pytest

from paper_1611_05984_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _domain(nx, ny, amp=0.03, dx=0.05, **params):
    """A sloping basin with a bank that dries, and a hump of water in motion."""
    from paper_1611_05984_amd import wavestep as ws
    X = np.arange(nx + 1)[None, :] / nx
    Y = np.arange(ny + 1)[:, None] / ny
    z = -0.5 + 0.1 * np.sin(7 * X + 5 * Y)
    z = np.where((X > 0.6) & (Y > 0.6), z + 0.45, z)
    d = ws.Domain(nx, ny, dx, dx, wl.courant_dt(0.2, dx, 0.6), z, **params)
    x = (np.arange(nx) + 0.5)[None, :] / nx
    y = (np.arange(ny) + 0.5)[:, None] / ny
    zc = 0.25 * ((z[:-1, :-1] + z[:-1, 1:]) + (z[1:, :-1] + z[1:, 1:]))
    h = amp * np.exp(-((x - 0.4) ** 2 + (y - 0.4) ** 2) / 0.02)
    d.set_state(np.maximum(h, zc), 2.0 * h, -1.3 * h)
    return d


def _same(a, b, what=""):
    for x, y in zip(a.state_numpy(), b.state_numpy()):
        assert np.isfinite(x).all() and np.array_equal(x, y), what


@pytest.mark.parametrize("nx,ny,before", [(130, 77, 0), (33, 64, 1), (64, 33, 2)])
def test_tuning_leaves_later_model_changes_alone(nx, ny, before):
    """The autotuner's predictor trials write F*, G* into the history level
    the next step writes.  NLSW steps after it must leave that level zero, as
    without it: for the dispersive steps that follow, and for a checkpoint."""
    from paper_1611_05984_amd import wavestep as ws
    print("case: tune then NLSW %dx%d after %d steps" % (nx, ny, before), flush=True)
    runs = []
    for tuned in (False, True):
        d = _domain(nx, ny)
        if before:      # NLSW steps before the trials: their levels are known to be zero
            d.update(model=ws.NLSW)
            d.advance(before)
            d.update(model=ws.BSNQ)
        if tuned:
            d.tune()
        d.set_tuning(16, 128, ws.SOLVE_PCR)
        d.update(model=ws.NLSW)
        d.advance(4)
        snap = d.snapshot()
        d.update(model=ws.BSNQ)
        d.advance(3)
        r = _domain(nx, ny, model=ws.NLSW)
        r.restore(snap)
        r.advance(1)
        r.update(model=ws.BSNQ)
        r.advance(3)
        runs.append((d, r))
    _same(runs[0][0], runs[1][0], "steps after the model change")
    _same(runs[0][1], runs[1][1], "steps after a restore")


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("change", ["sponge", "terrain", "dt"])
def test_changes_leave_queued_steps_alone(model, change):
    """Boundary, terrain and time-step changes right after steps were queued
    on a stream that the null stream does not wait for, against the same with
    the GPU waited for before every call."""
    import torch
    from paper_1611_05984_amd import wavestep as ws
    print("case: %s behind queued steps, model %d" % (change, model), flush=True)
    st = torch.cuda.Stream()
    runs = []
    for wait in (True, False):
        d = _domain(1024, 700, model=model)
        d.set_boundary(ws.NORTH, ws.SPONGE, 30, sponge_reflect=0.3)
        torch.cuda.synchronize()
        pause = torch.cuda.synchronize if wait else (lambda: None)
        for k in range(3):
            d.advance(60, stream=st)
            pause()
            if change == "terrain":
                assert d.apply_edit(ws.EDIT_TERRAIN, 15.0 + 5 * k, 12.0, 0.05, 2.0, stream=st) == 0
                pause()
            if change == "dt":
                d.update(dt=d.g.dt * 0.9)       # on the current stream, not the steps'
                pause()
            else:
                d.set_boundary(ws.EAST, ws.SPONGE, 40 + 100 * k)
                d.set_boundary(ws.SOUTH, (ws.SPONGE, ws.SOLID)[k % 2], 25)
                pause()
        d.advance(4, stream=st)
        torch.cuda.synchronize()
        assert d.query()[2] == 0
        runs.append(d)
    _same(runs[0], runs[1], change)


@pytest.mark.parametrize("nx,ny,model", [(90, 50, 0), (600, 530, 0), (40, 2100, 0), (90, 50, 1)])
def test_boundary_change_on_a_running_domain(nx, ny, model):
    """Steps, new sponges, more steps; against a fresh domain that had those
    sponges from the start and took the state over; alone and in a batch."""
    from paper_1611_05984_amd import wavestep as ws
    print("case: sponges set on a running %dx%d model %d" % (nx, ny, model), flush=True)

    def sponges(d):
        d.set_boundary(ws.EAST, ws.SPONGE, 12)
        d.set_boundary(ws.SOUTH, ws.SPONGE, 9, sponge_reflect=0.2)
        d.set_boundary(ws.WEST, ws.SOLID)

    a, f, b = (_domain(nx, ny, model=model) for _ in range(3))
    sponges(f)
    B = ws.Batch(1)
    B.attach(b)
    for d in (a, b):
        d.set_boundary(ws.WEST, ws.SPONGE, 7)
    a.advance(5)
    B.advance(5)
    B.sync()
    f.restore(a.snapshot())
    sponges(a)
    sponges(b)
    a.advance(4)
    f.advance(4)
    B.advance(4)
    B.sync()
    _same(a, f, "fresh domain")
    _same(a, b, "batch")
    B.close()


@pytest.mark.parametrize("model", [0, 1])
def test_boundary_change_before_a_captured_call(model):
    """A boundary change, a capture of the next steps, the same steps eagerly
    before the capture ever ran, then the capture replayed between eager
    steps: three steps each time, after which all buffers have their roles
    again."""
    import torch
    from paper_1611_05984_amd import wavestep as ws
    print("case: capture behind a boundary change, model %d" % model, flush=True)
    a, r = _domain(200, 90, model=model), _domain(200, 90, model=model)
    for d in (a, r):
        d.advance(3)
        d.set_boundary(ws.EAST, ws.SPONGE, 30)
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        a.advance(3, stream=st)
    a.advance(3)
    r.advance(3)
    torch.cuda.synchronize()
    _same(a, r, "eager steps before the first replay")
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        r.advance(3)
        _same(a, r, "replay %d" % k)
        a.advance(3)
        r.advance(3)
        torch.cuda.synchronize()
        _same(a, r, "eager steps after replay %d" % k)


@pytest.mark.parametrize("ny,batched", [(20, False), (20, True), (2060, False)])
def test_terrain_edit_leaves_nothing_beyond_the_rows(ny, batched):
    """The field of cell depths is built in the memory of the corners before
    the last terrain edit, and its rows are padded with them.  Corners chosen
    so that four of them in a row (0, 1, 42, 6/7 m deep, B = 1/6, dx = 1 m),
    taken for cell depths, have a pivot of exactly zero; every cell is 21 m
    deep.  The solves must not see them: the Thomas path's result, within the
    bound the strategies are held to."""
    from paper_1611_05984_amd import wavestep as ws
    print("case: pads behind rows of 17 cells, ny %d" % ny, flush=True)
    nx = 17
    s = np.tile([0.0, 0.0, 0.0, 0.0, 1.0, 42.0, 6.0 / 7.0, 0.0], 3)[:nx + 1] - 21.0
    z = -(21.0 - np.where(np.arange(ny + 1)[:, None] % 2, -1.0, 1.0) * s[None, :])

    def make():
        d = ws.Domain(nx, ny, 1.0, 1.0, 0.005, z, Bcoef=1.0 / 6.0)
        assert d.apply_edit(ws.EDIT_WATER, 8.0, 9.0, 0.05, 3.0) == 0
        for _ in range(2):      # either of the two corner arrays may be the field's
            assert d.apply_edit(ws.EDIT_TERRAIN, 3.0, 15.0, 1e-3, 1.0) == 0
        return d

    a, t = make(), make()
    t.set_tuning(16, 128, ws.SOLVE_THOMAS)
    t.advance(6)
    if batched:
        B = ws.Batch(1)
        B.attach(a)
        B.advance(6)
        B.sync()
        B.close()
    else:
        a.advance(6)
    for x, y in zip(a.state_numpy(), t.state_numpy()):
        assert np.isfinite(x).all() and np.abs(x - y).max() <= 1e-6 * max(1.0, np.abs(y).max())
    assert a.query()[2] == 0


def test_a_tuned_choice_can_be_set_again():
    """What the autotuner and tuning() return, set again on the same or
    another domain, runs what it ran: the same bits, and no slower (twice as
    slow at 128 x 64 cells when a returned 8 set the strips to 8 rows and a
    default of 32 to 32)."""
    import time

    import torch
    from paper_1611_05984_amd import wavestep as ws

    def us(d):
        best = 1e9
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            d.advance(150)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / 150 * 1e6)
        return best

    d = [_domain(128, 64) for _ in range(4)]
    assert d[0].tuning() == (8, 128, ws.SOLVE_PCR, 0)
    d[1].set_tuning(*d[0].tuning())
    choice = d[2].tune()
    assert d[2].tuning() == choice
    d[3].set_tuning(*choice)
    for x in d:
        x.advance(9)
    _same(d[0], d[1])
    _same(d[2], d[3])
    t = [us(x) for x in d]
    print("  us a step: fresh %.1f, its tuning set %.1f; tuned %s %.1f, its choice set %.1f"
          % (t[0], t[1], choice, t[2], t[3]), flush=True)
    assert t[1] <= 1.4 * t[0] and t[3] <= 1.4 * t[2]
