"""Reverse step of the row march at the edges of its strips.

The tiled form of the adjoint differentiates the same links cell by cell and is
held to the oracle elsewhere; both forms are compared on FP64 handles, where their
sums differ in order only (1e-10 relative: some 1e5 terms of 1e-16 each, with
cancellation), and on FP32 handles at the 1e-3 bar of the adjoint's other tests.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RAIN = np.array([130.0]) * 1e-3 / 3600.0


@pytest.fixture(scope="module")
def fl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2302_08341_amd import flood
    flood.load_library()
    return flood


def _run(fl, ny, nx, edges, rb, kernel, ckpt, t_end=12.0, n_members=5):
    rng = np.random.default_rng(ny * 1000 + nx)
    dem = (0.02 * rng.uniform(0.0, 1.0, (ny, nx)) + 0.01 * np.arange(ny)[:, None]).astype(np.float32)
    cat = dict(dem=dem, manning=rng.uniform(0.02, 0.05, (ny, nx)).astype(np.float32), dx=3.0, edge_kind=edges,
               edge_slope=tuple(1e-3 * e for e in edges), n_members=n_members,
               n_scale=rng.uniform(0.8, 1.2, n_members), rain_mult=rng.uniform(0.5, 1.5, n_members),
               h0=rng.uniform(0.2, 0.4, (ny, nx)).astype(np.float32))
    g = np.array([[0, 0], [ny - 1, nx - 1], [ny // 2, nx // 2]], dtype=np.int32)
    e = fl.FloodEnsemble([cat], RAIN, rain_interval=3600.0, member_interleave=1, step_kernel=kernel, real_bytes=rb)
    obs = np.full((int(t_end / 4.0), 3), 0.35)
    return e.adjoint(0, t_end, 4.0, g, obs, ckpt_every=ckpt)


def _close(a, b, rtol):
    assert abs(a[0] - b[0]) <= rtol * abs(b[0])
    assert np.linalg.norm(a[1] - b[1]) <= rtol * np.linalg.norm(b[1])
    assert np.linalg.norm(a[2] - b[2]) <= rtol * np.linalg.norm(b[2])


@pytest.mark.parametrize("rb,rtol", [(8, 1e-10), (4, 1e-3)])
@pytest.mark.parametrize("edges", [(1, 1, 1, 1), (1, 0, 0, 1), (0, 1, 1, 0)])
@pytest.mark.parametrize("ny,nx", [(1, 4), (2, 8), (3, 124), (9, 128), (33, 252), (17, 372)])
def test_strips_of_the_reverse_step(fl, ny, nx, edges, rb, rtol):
    _close(_run(fl, ny, nx, edges, rb, 3, 100), _run(fl, ny, nx, edges, rb, 1, 100), rtol)


@pytest.mark.parametrize("rows", [1, 3, 8, 16])
def test_rows_per_strip(fl, monkeypatch, rows):
    # strips of any height, the last one partly filled, give the same gradients
    ref = _run(fl, 35, 128, (1, 1, 1, 1), 8, 3, 100)
    monkeypatch.setenv("FLOOD_ADJ_ROWS", str(rows))
    monkeypatch.setenv("FLOOD_ADJ_FROWS", str(rows))
    _close(_run(fl, 35, 128, (1, 1, 1, 1), 8, 3, 100), ref, 1e-10)


@pytest.mark.parametrize("ckpt", [1, 2, 3, 7, 8, 9, 17, 30, 45])
def test_ends_of_the_tape_segments(fl, ckpt):
    # wherever the segments end, the loss and the rain-multiplier gradients are those
    # of the whole window in one segment, bit for bit
    ref = _run(fl, 24, 64, (1, 1, 1, 1), 8, 3, 1000)
    got = _run(fl, 24, 64, (1, 1, 1, 1), 8, 3, ckpt)
    assert got[0] == ref[0]
    np.testing.assert_array_equal(got[2], ref[2])
    assert np.linalg.norm(got[1] - ref[1]) <= 1e-10 * np.linalg.norm(ref[1])
