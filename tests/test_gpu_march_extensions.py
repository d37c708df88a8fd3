"""Row march with inflow links and running maxima, with and without land cover.

The forms with running maxima have their own registers and their own code: states are the
same bits as without them, and the maxima are those of the depths after every step.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

RAIN = np.array([90.0, 40.0]) * 1e-3 / 3600.0


@pytest.fixture(scope="module")
def fl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2302_08341_amd import flood
    flood.load_library()
    return flood


def _catch(land):
    c = W.urban_catchment("ext", 45, 264, 3, W.seed_for(2, 95), n_gauges=2, with_inflow=True, with_land_cover=True)
    d = dict(dem=c.dem, manning=c.manning, dx=c.dx, edge_kind=c.edge_kind, edge_slope=c.edge_slope, n_members=3,
             n_scale=c.n_scale, rain_mult=c.rain_mult, inflow=c.inflow, inflow_q=c.inflow_q)
    if land:
        d.update(land_class=c.land_class, class_runoff=c.class_runoff, class_drain=c.class_drain, class_n=c.class_n,
                 drain=c.drain)
    return d


@pytest.mark.parametrize("batch", [16, 3])   # steps that plan themselves, steps planned by the planner
@pytest.mark.parametrize("nt", [0, 1])       # plain and non-temporal accesses
@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("land", [False, True])
def test_maxima_with_inflow_links(fl, monkeypatch, land, rb, nt, batch):
    monkeypatch.setenv("FLOOD_GRAPH_STEPS", str(batch))
    monkeypatch.setenv("FLOOD_MARCH_NT", str(nt))
    cat = _catch(land)
    plain = fl.FloodEnsemble([cat], RAIN, real_bytes=rb)
    kept = fl.FloodEnsemble([cat], RAIN, real_bytes=rb, track_peak=True)
    peak = [np.zeros((45, 264)) for _ in range(3)]
    for _ in range(14):
        kept.step_n(130.0, 1)
        peak = [np.maximum(p, kept.field(m)) for m, p in enumerate(peak)]
    for m in range(3):
        np.testing.assert_array_equal(kept.field(m, fl.FIELD_PEAK), peak[m])
    whole = fl.FloodEnsemble([cat], RAIN, real_bytes=rb, track_peak=True)
    for e in (plain, kept, whole):
        e.step(130.0)
    for m in range(3):
        for w in (fl.FIELD_H, fl.FIELD_QX, fl.FIELD_QY):
            np.testing.assert_array_equal(plain.field(m, w), kept.field(m, w))
        np.testing.assert_array_equal(whole.field(m, fl.FIELD_PEAK), kept.field(m, fl.FIELD_PEAK))
        assert (whole.field(m, fl.FIELD_PEAK) >= peak[m]).all() and whole.field(m, fl.FIELD_PEAK).max() > 0.0
