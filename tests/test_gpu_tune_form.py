"""A tuned schedule is reused for the candidates it was chosen among: a choice
made with an inflow (no tile waves) or a given block height does not serve a free
solve of the same shape, nor the other way round, and lines of a tune cache that
were written for other schedules are not used."""
import numpy as np
import pytest

from paper_1811_12391_amd import dctsn, inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dctsn.lib()
    yield


def _problem(nx, ny, nz):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, 2, 1)
    dirs, w = I.lq_quadrature(4)
    pos, axis = I.ring_sources(1, 360.0)
    return I.Problem("form", ph, xs, dirs, w, 1, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))


INFLOW = np.array([1.0, 2.0])


@pytest.mark.parametrize("grid", [(21, 35, 7), (33, 70, 18)])
@pytest.mark.parametrize("first", [dict(test_inflow=INFLOW), dict(sweep_bk=4), dict(sweep_sync=2)])
def test_restricted_tuning_is_not_reused(grid, first):
    prob = _problem(*grid)
    kw = dict(precision="fp32", fixed_iters=np.array([2, 2], dtype=np.int32), autotune=True)
    s = dctsn.Solver(prob)
    try:
        a = s.solve(**kw, **first)
        free = s.solve(**kw)
        print(f"[form] {grid} {sorted(first)}: {a.sweep_bk}:{a.sweep_sync}, free {free.sweep_bk}:{free.sweep_sync}", flush=True)
        assert a.tune_ms > 0 and free.tune_ms > 0
        # both choices are kept
        b, c = s.solve(**kw, **first), s.solve(**kw)
        assert b.tune_ms == 0 and (b.sweep_bk, b.sweep_sync) == (a.sweep_bk, a.sweep_sync)
        assert c.tune_ms == 0 and (c.sweep_bk, c.sweep_sync) == (free.sweep_bk, free.sweep_sync)
    finally:
        s.close()


def test_cache_lines_of_other_schedules(tmp_path, monkeypatch):
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("DCT_TUNE_CACHE", str(path))
    prob = _problem(33, 70, 18)
    kw = dict(precision="fp32", fixed_iters=np.array([2, 2], dtype=np.int32), autotune=True)
    s = dctsn.Solver(prob)
    s.solve(**kw)
    s.close()
    line = path.read_text().split()
    # as a build with other layouts and couplings wrote it: no version, or another one
    for old in (line[:14], line[:14] + ["1", line[15]]):
        path.write_text(" ".join(old) + "\n")
        s = dctsn.Solver(prob)
        try:
            assert s.solve(**kw).tune_ms > 0
        finally:
            s.close()
    assert path.read_text().splitlines()[-1].split()[14:] == line[14:]
    s = dctsn.Solver(prob)
    try:
        assert s.solve(**kw).tune_ms == 0
        assert s.solve(**dict(kw, test_inflow=INFLOW)).tune_ms > 0
    finally:
        s.close()


def test_forced_tile_waves_with_inflow():
    """Coupling 4 asked for with an inflow runs as the barrier coupling, tuned as
    untuned."""
    prob = _problem(21, 35, 7)
    kw = dict(precision="fp64", fixed_iters=np.array([2, 2], dtype=np.int32), sweep_sync=4, test_inflow=INFLOW)
    s = dctsn.Solver(prob)
    try:
        a = s.solve(**kw)
        d = s.dose()
        b = s.solve(autotune=True, **kw)
        assert (a.sweep_sync, b.sweep_sync) == (2, 2) and np.array_equal(s.dose(), d)
    finally:
        s.close()
