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
@pytest.mark.parametrize("plain,land", [([(53, 72, 4)], [(40, 264, 2)]), ([(33, 64, 3), (45, 80, 1)], [(70, 128, 2), (17, 28, 5)])])
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


class _Batch:
    """Catchments of one handle, each with its own parameters."""

    def __init__(self, fl, cats, rb, track_peak):
        self.fl, self.cats = fl, cats
        grids = [fl.make_grid(c["dem"], c["manning"], c["dx"], c["edge_kind"], c["edge_slope"],
                              land_class=c.get("land_class")) for c in cats]
        params = [fl.make_params(RAIN, real_bytes=rb, track_peak=p, class_runoff=c.get("class_runoff"),
                                 class_drain=c.get("class_drain"), member_class_n=c.get("class_n"),
                                 member_drain=c.get("drain")) for c, p in zip(cats, track_peak)]
        self.h = fl.flood_create_batch(grids, params, [c["n_members"] for c in cats], [c["n_scale"] for c in cats],
                                       [c["rain_mult"] for c in cats])

    def field(self, m, w, i):
        ny, nx = self.cats[i]["dem"].shape
        shape = {self.fl.FIELD_QX: (ny, nx + 1), self.fl.FIELD_QY: (ny + 1, nx)}.get(w, (ny, nx))
        return self.fl.flood_get_field(self.h, i, m, w, shape)

    def ledger(self, i):
        return self.fl.flood_get_ledger(self.h, i, self.cats[i]["n_members"])


# ragged rows, whole vectors, and land cover beside plain catchments; few wavefronts and more
@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("shapes,land", [([(21, 37, 2), (34, 65, 3)], (0, 0)), ([(300, 257, 16), (90, 1030, 16)], (0, 0)),
                                         ([(300, 512, 8), (260, 512, 8), (250, 512, 6)], (0, 0, 0)),
                                         ([(41, 260, 2), (38, 128, 3), (25, 64, 2)], (0, 1, 1))])
@pytest.mark.parametrize("first", [0, 1])
def test_maxima_of_some_catchments(fl, shapes, land, rb, first):
    track = [(i + first) % 2 for i in range(len(shapes))]
    cats = [_catch(*s, seed=80 + i, land=bool(k)) for i, (s, k) in enumerate(zip(shapes, land))]
    both = _Batch(fl, cats, rb, track)
    for t in (20.0, 45.0):
        fl.flood_step(both.h, t)
    for i, c in enumerate(cats):
        alone = fl.FloodEnsemble([c], RAIN, real_bytes=rb, track_peak=bool(track[i]))
        alone.step(20.0)
        alone.step(45.0)
        _same_catchment(fl, both, i, alone, c["n_members"], peak=bool(track[i]))
        if track[i]:
            assert both.field(0, fl.FIELD_PEAK, i).max() > 0.0
        else:
            with pytest.raises(fl.FloodError) as ex:
                both.field(0, fl.FIELD_PEAK, i)
            assert ex.value.status == fl.FLOOD_ESTATE
    fl.flood_destroy(both.h)


@pytest.mark.parametrize("rb", [4, 8])
def test_a_plain_handle_leaves_land_cover_its_own_strips(fl, monkeypatch, rb):
    # strips measured for plain catchments (one row tall on small grids) are not those of land
    # cover, whose drained volume is summed over rows of a strip
    plain, land = _catch(61, 88, 3, seed=91), _catch(61, 88, 3, seed=91, land=True)
    fl.FloodEnsemble([plain], RAIN, real_bytes=rb).step(10.0)
    after = fl.FloodEnsemble([land], RAIN, real_bytes=rb)
    monkeypatch.setenv("FLOOD_AUTOTUNE", "0")
    alone = fl.FloodEnsemble([land], RAIN, real_bytes=rb)
    assert fl.flood_get_march_rows(after.h, 0) % 4 == 0 or fl.flood_get_march_rows(after.h, 0) == 61
    for e in (after, alone):
        e.step(400.0)
    np.testing.assert_array_equal(after.field(1), alone.field(1))
    assert (alone.ledger()["drain"] > 0.0).all()
    np.testing.assert_allclose(after.ledger()["drain"], alone.ledger()["drain"], rtol=1e-12)


def test_a_handle_that_names_its_kernel_measures_it(fl):
    c = _catch(61, 92, 3, seed=92)
    open_ = fl.FloodEnsemble([c], RAIN, real_bytes=4)
    assert open_.config()["step_kernel"] == 3
    named = fl.FloodEnsemble([c], RAIN, real_bytes=4, step_kernel=2)
    assert named.config()["step_kernel"] == 2
    assert fl.flood_get_march_rows(named.h, 0) >= 8
