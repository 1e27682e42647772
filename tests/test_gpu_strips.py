"""Strip heights the library picks by itself (1, 2 or 8 rows by the number
of waves a grid gives) against heights the caller sets: the same bits, alone
and in a batch, for every kind of boundary and both friction laws (whose
roundings must not depend on how far the row loop is unrolled)."""
import numpy as np
import pytest

from paper_1611_05984_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _make(nx, ny, **params):
    from paper_1611_05984_amd import wavestep as ws
    w = wl.config2(nx=nx, ny=ny, seed=nx + ny)
    d = ws.Domain(nx, ny, w.dx, w.dy, w.dt, w.z, **params)
    side = w.sides[wl.WEST]
    d.set_boundary(ws.WEST, ws.WAVES, 2, side.amp, side.period, [0.3], [0.1])
    d.set_boundary(ws.NORTH, ws.SPONGE, 6)
    assert d.apply_edit(ws.EDIT_WATER, 0.3 * nx * w.dx, 0.5 * ny * w.dy, 0.05, 8 * w.dx) == 0
    return d


def _same(a, b, what):
    for x, y in zip(a.state_numpy(), b.state_numpy()):
        assert np.isfinite(x).all() and np.array_equal(x, y), what


# strips of 62 columns: ceil(nx / 62) * ceil(ny / rows) waves; 1 row up to 4096, 2 up to 72000
@pytest.mark.parametrize("nx,ny,params", [
    (62, 9, dict(friction=2, friction_coef=0.03)),     # 1 row, one whole strip
    (63, 17, dict(friction=1, friction_coef=0.01)),    # 1 row, a strip of one column
    (310, 819, dict()),                                # 4095 waves: the last of 1 row
    (310, 821, dict(friction=2, friction_coef=0.03)),  # 2 rows, an odd last strip
    (992, 417, dict(friction=1, friction_coef=0.01)),  # 2 rows, a last strip of one row
    (3100, 2883, dict(n_corr=1)),                      # 8 rows
])
def test_own_heights_equal_set_heights(nx, ny, params):
    from paper_1611_05984_amd import wavestep as ws
    print("case: %dx%d %s" % (nx, ny, params), flush=True)
    own = _make(nx, ny, **params)
    own.advance(9)
    for rows, crows in ((8, 0), (24, 16)):
        d = _make(nx, ny, **params)
        d.set_tuning(rows, 128, ws.SOLVE_PCR, crows)
        d.advance(9)
        _same(own, d, (nx, ny, rows, crows))
        d.close()
    b = _make(nx, ny, **params)
    B = ws.Batch(1)
    B.attach(b)
    B.advance(9)
    B.sync()
    _same(own, b, (nx, ny, "batch"))
    B.close()
