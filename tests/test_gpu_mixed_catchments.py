"""Catchments of different kinds in one handle against one handle for each.

A catchment's step does not depend on the others: every field, clock and step count
is the same bits.  The ledger's volumes are FP64 sums whose order follows the
launch's geometry (1e-12 relative).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

RAIN = np.array([130.0, 60.0]) * 1e-3 / 3600.0


@pytest.fixture(scope="module")
def fl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2302_08341_amd import flood
    flood.load_library()
    return flood


def _catch(ny, nx, n_members, seed, land=False):
    c = W.urban_catchment("mixed%d" % seed, ny, nx, n_members, W.seed_for(2, seed), n_gauges=2, with_land_cover=land)
    d = dict(dem=c.dem, manning=c.manning, dx=c.dx, edge_kind=c.edge_kind, edge_slope=c.edge_slope,
             n_members=n_members, n_scale=c.n_scale, rain_mult=c.rain_mult)
    if land:
        d.update(land_class=c.land_class, class_runoff=c.class_runoff, class_drain=c.class_drain, class_n=c.class_n,
                 drain=c.drain)
    return d


def _same_catchment(fl, both, i, alone, n_members, peak=False):
    which = (fl.FIELD_H, fl.FIELD_QX, fl.FIELD_QY) + ((fl.FIELD_PEAK,) if peak else ())
    for m in range(n_members):
        for w in which:
            np.testing.assert_array_equal(both.field(m, w, i), alone.field(m, w))
    la, lb = both.ledger(i), alone.ledger()
    for k in ("rain_in", "t", "steps"):
        np.testing.assert_array_equal(la[k], lb[k])
    for k in ("storage", "outflow", "drain"):
        np.testing.assert_allclose(la[k], lb[k], rtol=1e-12)


@pytest.mark.parametrize("batch", [16, 3])      # steps that plan themselves, steps planned by the planner
@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("plain,land", [([(54, 76, 4)], [(40, 264, 2)]), ([(33, 64, 3), (45, 80, 1)], [(70, 128, 2), (17, 28, 5)])])
def test_catchments_with_and_without_land_cover(fl, monkeypatch, plain, land, rb, batch):
    monkeypatch.setenv("FLOOD_GRAPH_STEPS", str(batch))
    cats, kinds = [], []
    for i in range(len(plain)):
        for k in (len(plain) > 1, len(plain) == 1):      # land cover first, or last
            cats.append(_catch(*(land if k else plain)[i], seed=70 + i, land=k))
            kinds.append(k)
    both = fl.FloodEnsemble(cats, RAIN, real_bytes=rb, track_peak=True)
    both.step(200.0)
    both.step(420.0)
    for i, c in enumerate(cats):
        alone = fl.FloodEnsemble([c], RAIN, real_bytes=rb, track_peak=True)
        alone.step(200.0)
        alone.step(420.0)
        _same_catchment(fl, both, i, alone, c["n_members"], peak=True)
        assert (both.ledger(i)["drain"] > 0.0).any() == kinds[i]
