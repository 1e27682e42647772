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
