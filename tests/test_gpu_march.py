"""Vectorised row march at the edges of its strips, lanes and batches.

The tiled kernel (step_kernel 1) evaluates the same link functions per cell and is
held to the oracle elsewhere; every path of the row march must give its bits.
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


def _catch(ny, nx, n_members, edges=(1, 1, 1, 1), seed=11):
    rng = np.random.default_rng(seed)
    dem = (0.02 * rng.uniform(0.0, 1.0, (ny, nx)) + 0.01 * np.arange(ny)[:, None]).astype(np.float32)
    return dict(dem=dem, manning=rng.uniform(0.02, 0.05, (ny, nx)).astype(np.float32), dx=3.0, edge_kind=edges,
                edge_slope=tuple(1e-3 * e for e in edges), n_members=n_members, n_scale=rng.uniform(0.8, 1.2, n_members),
                rain_mult=rng.uniform(0.5, 1.5, n_members), h0=rng.uniform(0.0, 0.3, (ny, nx)).astype(np.float32))


def _same(fl, cat, t_end, **kw):
    a = fl.FloodEnsemble([cat], RAIN, member_interleave=1, step_kernel=1, track_peak=True, real_bytes=kw["real_bytes"])
    b = fl.FloodEnsemble([cat], RAIN, member_interleave=1, track_peak=True, **kw)
    a.step(t_end)
    b.step(t_end)
    assert b.config()["step_kernel"] == 3
    for m in range(cat["n_members"]):
        for w in (fl.FIELD_H, fl.FIELD_QX, fl.FIELD_QY, fl.FIELD_PEAK):
            np.testing.assert_array_equal(a.field(m, w), b.field(m, w))
    la, lb = a.ledger(), b.ledger()
    for k in ("rain_in", "t", "steps"):
        np.testing.assert_array_equal(la[k], lb[k])
    for k in ("outflow", "storage"):     # FP64 sums in another order
        np.testing.assert_allclose(la[k], lb[k], rtol=1e-12)


@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("ny,nx,rows", [(5, 1, 2), (3, 3, 64), (70, 255, 7), (130, 257, 100), (66, 259, 64), (131, 130, 65)])
def test_rows_of_any_length(fl, monkeypatch, rb, ny, nx, rows):
    # without the tuner a handle that names no kernel takes the row march, whatever its row length
    monkeypatch.setenv("FLOOD_AUTOTUNE", "0")
    _same(fl, _catch(ny, nx, 2), 20.0, real_bytes=rb, march_rows=rows)


@pytest.mark.parametrize("edges", [(1, 0, 0, 1), (0, 1, 1, 0)])
@pytest.mark.parametrize("rows", [1, 63, 64, 65, 129])
def test_tall_strips_and_edges(fl, edges, rows):
    # the domain's west and east edge links are kept for 64 rows at a time
    _same(fl, _catch(130, 512, 2, edges), 15.0, real_bytes=4, step_kernel=3, march_rows=rows)


def test_stores_under_load(fl):
    # 1024 columns x 1024 rows x 4 members: enough waves in flight that a store's data
    # register can still be unread when the next instruction issues; the adjoint's recording
    # forward writes blocks that nothing else rewrites
    c = W.urban_catchment("march", 1024, 1024, 4, 123, n_gauges=4)
    cat = dict(dem=c.dem, manning=c.manning, dx=c.dx, edge_kind=c.edge_kind, edge_slope=c.edge_slope, n_members=4,
               n_scale=c.n_scale, rain_mult=c.rain_mult)
    ens = [fl.FloodEnsemble([cat], RAIN, step_kernel=sk) for sk in (1, 3)]
    loss = []
    for e in ens:
        e.step(50.0)
        loss.append(e.adjoint(0, 60.0, 10.0, c.gauges, np.full((1, 4), 0.05), 100)[0])
    assert loss[0] == loss[1]
    for m in range(4):
        for w in (fl.FIELD_H, fl.FIELD_QX, fl.FIELD_QY):
            np.testing.assert_array_equal(ens[0].field(m, w), ens[1].field(m, w))


@pytest.mark.parametrize("rb", [4, 8])
def test_steps_that_plan_themselves(fl, monkeypatch, rb):
    # batches of three steps are planned by the planner kernel, batches of four or sixteen by
    # the steps: the same clocks, logs, ledgers and states, with bounded calls, calls that move
    # nothing, rain-block edges, a member that faults and catchments of different sizes
    cats = [_catch(40, 128, 3, seed=5), _catch(21, 64, 2, (0, 1, 0, 1), seed=6)]

    def run(batch):
        monkeypatch.setenv("FLOOD_GRAPH_STEPS", str(batch))
        e = fl.FloodEnsemble(cats, RAIN, rain_interval=7.0, real_bytes=rb, step_kernel=3, march_rows=8)
        e.log_steps(256)
        e.step_n(30.0, 5)
        e.step(3.0)
        e.step(9.5)
        h = e.field(1)
        h[3, 3] = 3e38 if rb == 4 else 1e300        # Eq. 4 no longer advances this member's clock
        e.set_state(1, h, e.field(1, fl.FIELD_QX), e.field(1, fl.FIELD_QY), 9.5)
        try:
            e.step(25.0)
            status = 0
        except fl.FloodError as err:
            status = err.status
        out = [status]
        for c in range(2):
            led = e.ledger(c)
            out += [led[k] for k in ("rain_in", "t", "steps", "inflow", "drain")] + list(e.step_log(c))
            out += [e.field(m, w, c) for m in range(cats[c]["n_members"]) for w in (0, 1, 2)]
        return out

    ref = run(3)
    assert ref[0] == fl.FLOOD_ENUMERIC
    for batch in (4, 16):
        got = run(batch)
        for a, b in zip(ref, got):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("ny,nx,rows", [(1, 1, 1), (5, 63, 1), (6, 64, 2), (7, 65, 3), (131, 129, 8), (66, 200, 64)])
def test_strips_of_one_cell_a_lane(fl, monkeypatch, rb, ny, nx, rows):
    # few wavefronts: strips of 64 cells, whose maxima a workgroup sends together
    monkeypatch.setenv("FLOOD_AUTOTUNE", "0")
    _same(fl, _catch(ny, nx, 3), 20.0, real_bytes=rb, march_rows=rows)


@pytest.mark.parametrize("rb", [4, 8])
@pytest.mark.parametrize("ny,nx,members,rows", [(5, 1, 400, 2), (70, 255, 30, 7), (66, 259, 20, 64)])
def test_ragged_rows_of_many_members(fl, monkeypatch, rb, ny, nx, members, rows):
    # enough wavefronts: strips of whole vectors, the last of a row cut short
    monkeypatch.setenv("FLOOD_AUTOTUNE", "0")
    _same(fl, _catch(ny, nx, members), 10.0, real_bytes=rb, march_rows=rows)


@pytest.mark.parametrize("rb", [4, 8])
def test_members_that_end_at_different_times_in_narrow_strips(fl, monkeypatch, rb):
    # wavefronts of members past their end leave workgroups whose others go on
    monkeypatch.setenv("FLOOD_AUTOTUNE", "0")
    cat = _catch(9, 130, 6)
    cat["rain_mult"] = np.array([0.0, 40.0, 0.1, 20.0, 5.0, 1.0])
    _same(fl, cat, 60.0, real_bytes=rb, march_rows=2)


@pytest.mark.parametrize("rb", [4, 8])
def test_a_short_step_at_a_block_edge_is_no_estimate(fl, rb):
    # the first batch of 16 ends with a step of 1 ms up to the edge of a rain block; the 3 steps
    # after it take one batch of 4, not two of 16
    e = fl.FloodEnsemble([_catch(40, 128, 3)], RAIN, rain_interval=15.001, dt_fixed=1.0, real_bytes=rb, step_kernel=3,
                         march_rows=8)
    fl.flood_timing(e.h, fl.TIMING_BATCH)
    e.step(18.0)
    assert (e.ledger()["steps"] == 19).all()
    assert fl.flood_get_timing(e.h)[1] == 20
