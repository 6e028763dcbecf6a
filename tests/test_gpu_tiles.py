"""Tile-wave sweeps (coupling 4): every wave sweeps tiles of 16 y rows x 4 z
layers.  Each cell's arithmetic is that of the other schedules, so moments,
dose and iteration counts equal the barrier coupling's bit for bit on every
grid: rows shorter than a tile's skew, one row or one layer, partial tiles in
y and z, several tiles per wave, grids of several 64 x 16 blocks."""
import sys

import numpy as np
import pytest

from paper_1811_12391_amd import dctsn, inputs as I

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dctsn.lib()
    yield


def _problem(nx, ny, nz, sources=1, sn=4, L=1, groups=3):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, groups, L)
    dirs, w = I.lq_quadrature(sn)
    pos, axis = I.ring_sources(sources, 360.0 / sources)
    return I.Problem("tiles", ph, xs, dirs, w, L, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))


def _tile_kw(prob):
    """Small one-block grids take the barrier coupling untuned: ask for tiles."""
    ph = prob.phantom
    return dict(sweep_bk=16, sweep_sync=4) if ph.ny <= 64 and ph.nz <= 16 else {}


def _run(prob, **kw):
    s = dctsn.Solver(prob)
    try:
        st = s.solve(**kw)
        return st, s.dose(), s.moments()
    finally:
        s.close()


# the last two numbers: sources and directions S_N, which set the y streams
GRIDS = [(1, 1, 1, 1, 4), (5, 1, 3, 1, 4), (13, 11, 5, 1, 4), (19, 16, 4, 1, 4), (32, 17, 9, 1, 4), (31, 33, 16, 2, 4),
         (64, 15, 1, 1, 4), (40, 64, 13, 1, 6), (24, 61, 16, 40, 6), (64, 64, 16, 36, 6), (33, 70, 18, 1, 4),
         (20, 130, 33, 1, 4), (48, 80, 64, 1, 4), (30, 100, 20, 24, 4)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("grid", GRIDS)
def test_tiles_bitwise(grid, prec):
    nx, ny, nz, B, sn = grid
    prob = _problem(nx, ny, nz, B, sn)
    fi = np.full(prob.G, 3, dtype=np.int32)
    _say(f"[tiles] {grid} {prec}")
    for fix in (True, False):
        st0, d0, m0 = _run(prob, precision=prec, fixed_iters=fi, fixup=fix, sweep_bk=16, sweep_sync=2)
        st, d, m = _run(prob, precision=prec, fixed_iters=fi, fixup=fix, **_tile_kw(prob))
        assert (st0.sweep_sync, st.sweep_sync) == (2, 4)
        assert np.array_equal(m, m0) and np.array_equal(d, d0) and np.array_equal(st.eps, st0.eps)
        # the boundary outflows are summed in another order (in FP32 within a row)
        assert np.allclose(st.balance, st0.balance, rtol=1e-11 if prec == "fp64" else 1e-5, atol=1e-300)


def test_tiles_inflow_and_balance():
    """Vacuum boundaries, converged in FP64: bitwise, and the balance closes; an
    inflow through the faces takes another schedule."""
    prob = _problem(21, 35, 7)
    for infl, sync in ((None, 4), (np.linspace(1.0, 2.0, prob.G), 2)):
        kw = dict(precision="fp64", tol=1e-12, test_inflow=infl)
        st0, d0, _ = _run(prob, sweep_bk=16, sweep_sync=2, **kw)
        st, d, _ = _run(prob, **_tile_kw(prob), **kw)
        assert st.sweep_sync == sync and np.array_equal(d, d0) and np.array_equal(st.iters, st0.iters)
        P, R, Lk = st.balance[0].T
        assert np.max(np.abs(P - R - Lk) / P) < 1e-9


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("grid", [(13, 11, 5), (40, 45, 13), (36, 70, 18)])
def test_tiles_adjoint(grid, prec):
    """Kept fluxes and fixup sets, and the transposed sweeps: the gradients are
    those of the barrier coupling up to the order of the ray atomics."""
    prob = _problem(*grid)
    C = prob.phantom.C
    roi = np.random.default_rng(3).random(C)
    fi = np.full(prob.G, 4, dtype=np.int32)
    res = []
    for kw in (dict(sweep_bk=16, sweep_sync=2), _tile_kw(prob)):
        s = dctsn.Solver(prob)
        try:
            st = s.solve(precision=prec, fixed_iters=fi, keep_adjoint=True, **kw)
            res.append((st.sweep_sync, s.dose(), s.adjoint(roi, fixed_iters=fi)))
        finally:
            s.close()
    assert (res[0][0], res[1][0]) == (2, 4)
    assert np.array_equal(res[0][1], res[1][1])
    a, b = res[0][2], res[1][2]
    assert a.R == b.R and np.array_equal(a.eps, b.eps)
    assert np.allclose(a.d_density, b.d_density, rtol=0, atol=1e-12 * np.abs(a.d_density).max())
    assert np.allclose(a.d_group_w, b.d_group_w, rtol=1e-12, atol=0)


@pytest.mark.parametrize("prec", ["fp32", "fp64", "fp32_bf16map"])
@pytest.mark.parametrize("nx,ny,nz,src,sn", [(40, 64, 13, 1, 6), (33, 70, 18, 1, 4), (24, 61, 16, 9, 6)])
def test_tuned_equals_untuned(nx, ny, nz, src, sn, prec):
    """The tuner times schedules in both tile widths of the layouts; the solve
    that follows, and one that takes its choice from the start, equal the
    barrier coupling's, also with acceleration (another reader of the layouts)."""
    prob = _problem(nx, ny, nz, src, sn)
    fi = np.array([2, 3, 1], dtype=np.int32)
    for kw in (dict(fixed_iters=fi), dict(tol=1e-3, max_iter=30, allow_notconv=True, accel_depth=2)):
        st0, d0, m0 = _run(prob, precision=prec, sweep_sync=2, **kw)
        s = dctsn.Solver(prob)
        try:
            for tune in (True, False):
                st = s.solve(precision=prec, autotune=tune, **kw)
                _say(f"[tuned] {nx}x{ny}x{nz} {prec} autotune {tune}: coupling {st.sweep_sync}")
                assert np.array_equal(st.iters, st0.iters)
                assert np.array_equal(s.dose(), d0) and np.array_equal(s.moments(), m0)
        finally:
            s.close()
