"""Drained volume of the land-cover ledger: how many single-precision terms a partial sum has.

On a flat walled pond of one draining class every cell loses the same depth d in every
step, so a lane's partial sum over R rows of 4 cells is 4 R additions of d and the
ledger is a whole number of such sums (added in FP64: 1e-12).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2302_08341_amd import flood
    flood.load_library()
    return flood


@pytest.mark.parametrize("ny,nx,members,rows", [(64, 96, 4, 4), (248, 400, 60, 4), (400, 512, 64, 4), (512, 1024, 40, 8)])
def test_rows_of_a_partial_sum(fl, ny, nx, members, rows):
    rate, steps, dx = 2.7182817e-6, 3, 3.0
    cat = dict(dem=np.zeros((ny, nx), np.float32), manning=np.full((ny, nx), 0.03, np.float32), dx=dx,
               edge_kind=(0, 0, 0, 0), edge_slope=(0.0,) * 4, n_members=members, h0=np.full((ny, nx), 0.5, np.float32),
               land_class=np.zeros((ny, nx), np.uint8), class_runoff=np.ones(1), class_drain=np.ones(1, np.int32),
               class_n=np.full((members, 1), 0.03), drain=np.full(members, rate))
    e = fl.FloodEnsemble([cat], np.zeros(1), rain_interval=1000.0, dt_fixed=1.0, real_bytes=4)
    e.step(float(steps))
    assert fl.flood_get_march_rows(e.h, 0) % rows == 0
    d = np.float32(rate)
    part = {r: np.float64(np.add.accumulate(np.full(4 * r, d, np.float32), dtype=np.float32)[-1]) / (4 * r) for r in (4, 8, 16)}
    assert abs(part[4] / part[8] - 1.0) > 1e-9 and abs(part[8] / part[16] - 1.0) > 1e-9   # the sums tell the rows apart
    np.testing.assert_allclose(e.ledger()["drain"], steps * ny * nx * part[rows] * dx * dx, rtol=1e-12)
