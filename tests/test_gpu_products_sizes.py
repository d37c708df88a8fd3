"""Ensemble products over the member counts at which the kernel changes its form:
sorted values in registers up to 16, 32, 64 and 128 members (64 in FP64), candidates
shared by four wavefronts past them.  Against the oracle, whose weights are summed in
the same order, so both maps agree bit for bit.
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


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


PCT = (0.5, 0.1, 1.0, 0.25, 0.9, 1e-12, 0.75, 0.3)


@pytest.mark.parametrize("rb,mi", [(4, 1), (4, 4), (8, 1), (8, 2)])
@pytest.mark.parametrize("N,n_pct", [(1, 1), (15, 2), (16, 3), (17, 4), (33, 8), (64, 5), (65, 3), (128, 2), (129, 1),
                                     (200, 3)])
def test_products_of_any_member_count(fl, orc, N, n_pct, rb, mi):
    ny, nx = 9, 23                       # 207 cells: three whole wavefronts and 15 cells
    rng = np.random.default_rng(N + rb)
    cat = dict(dem=np.zeros((ny, nx), np.float32), manning=np.full((ny, nx), 0.03, np.float32), dx=2.0,
               edge_kind=(0, 0, 0, 0), edge_slope=(0.0,) * 4, n_members=N, n_scale=np.ones(N), rain_mult=np.ones(N),
               h0=np.zeros((ny, nx), np.float32))
    e = fl.FloodEnsemble([cat], np.array([1e-6]), real_bytes=rb, member_interleave=mi, track_peak=True)
    # values with ties and dry cells
    h = np.round(rng.uniform(-0.1, 1.0, (N, ny, nx)), 2).clip(min=0.0).astype(np.float32).astype(np.float64)
    for m in range(N):
        e.set_state(m, h[m], np.zeros((ny, nx + 1)), np.zeros((ny + 1, nx)), 0.0)
    for w in (None, rng.integers(0, 3, N) + (np.arange(N) == 0), rng.uniform(0.0, 1.0, N)):
        wf = None if w is None else np.asarray(w, dtype=np.float64)
        prob, pc = e.products(0.3, PCT[:n_pct], weights=wf)
        peaks = np.stack([e.field(m, fl.FIELD_PEAK) for m in range(N)])
        rp, rpc = orc.ensemble_products(peaks, 0.3, PCT[:n_pct], weights=wf)
        np.testing.assert_array_equal(prob, rp)
        np.testing.assert_array_equal(pc, np.stack(rpc))


@pytest.mark.parametrize("ny,nx", [(512, 512), (513, 512), (1100, 1000)])
def test_fields_larger_than_the_staging_slots(fl, ny, nx):
    # a slot holds 512 x 512 values, the ring three slots
    rng = np.random.default_rng(ny)
    cat = dict(dem=np.zeros((ny, nx), np.float32), manning=np.full((ny, nx), 0.03, np.float32), dx=2.0,
               edge_kind=(1, 1, 1, 1), edge_slope=(1e-3,) * 4, n_members=2, n_scale=np.ones(2), rain_mult=np.ones(2),
               h0=np.zeros((ny, nx), np.float32))
    e = fl.FloodEnsemble([cat], np.array([1e-6]), real_bytes=8, member_interleave=1, track_peak=True)
    h, qx, qy = rng.uniform(0, 1, (ny, nx)), rng.uniform(0, 1, (ny, nx + 1)), rng.uniform(0, 1, (ny + 1, nx))
    e.set_state(1, h, qx, qy, 0.0)
    for which, want in ((fl.FIELD_H, h), (fl.FIELD_QX, qx), (fl.FIELD_QY, qy), (fl.FIELD_PEAK, h)):
        np.testing.assert_array_equal(e.field(1, which), want)
    prob, pc = e.products(0.5, PCT[:3])
    np.testing.assert_array_equal(prob, (h >= 0.5) / 2.0)
    np.testing.assert_array_equal(pc[2], h)          # p = 1: the larger of 0 and h
    np.testing.assert_array_equal(pc[1], 0.0 * h)
