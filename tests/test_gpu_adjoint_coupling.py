"""The transposed sweeps' own coupling: after layered waves (which have no
transposed form), after tile waves that were asked for, and after tile waves
that tuning or the default chose; every one gives the oracle's gradient, and the
choices give one another's up to the order of the ray atomics."""
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


def _close(got, ref, tol):
    assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref))


def test_adjoint_after_layered_waves():
    import oracle

    prob = I.make_problem("tiny_abd")
    roi = np.random.default_rng(7).random(prob.phantom.C)
    fwd = oracle.solve_problem(prob, tol=1e-10)
    fi = fwd.iters.max(0).astype(np.int32)
    ref = oracle.adjoint_problem(prob, roi, fixed_iters=fi, fixed_iters_adj=fi)
    for sync in (5, 4, 2):
        s = dctsn.Solver(prob)
        try:
            st = s.solve(precision="fp64", fixed_iters=fi, keep_adjoint=True, sweep_bk=16, sweep_sync=sync)
            assert st.sweep_sync == sync
            a = s.adjoint(roi, fixed_iters=fi)
        finally:
            s.close()
        assert abs(a.R - ref.R) <= 1e-10 * abs(ref.R)
        _close(a.d_density, ref.d_density, 1e-10)
        _close(a.d_group_w, ref.d_group_w, 1e-10)


# one block with and without the barrier coupling first, several blocks
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz", [(24, 20, 9), (20, 33, 16), (33, 70, 18), (3, 80, 5)])
def test_choices_agree(nx, ny, nz, prec):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, 2, 1)
    dirs, w = I.lq_quadrature(4)
    pos, axis = I.ring_sources(1, 360.0)
    prob = I.Problem("choice", ph, xs, dirs, w, 1, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))
    roi = np.random.default_rng(3).random(ph.C)
    fi = np.array([4, 3], dtype=np.int32)
    one = ny <= 64 and nz <= 16
    forms = [dict(sweep_bk=16, sweep_sync=2), dict(), dict(autotune=True)]
    if one:
        forms += [dict(sweep_bk=16, sweep_sync=4), dict(sweep_bk=16, sweep_sync=5)]
    res = []
    for kw in forms:
        s = dctsn.Solver(prob)
        try:
            st = s.solve(precision=prec, fixed_iters=fi, keep_adjoint=True, **kw)
            res.append((s.dose(), s.adjoint(roi, fixed_iters=fi)))
            print(f"[choice] {nx}x{ny}x{nz} {prec} {kw}: coupling {st.sweep_sync}", flush=True)
        finally:
            s.close()
    d0, a = res[0]
    for d, b in res[1:]:
        assert np.array_equal(d, d0) and a.R == b.R and np.array_equal(a.eps, b.eps)
        _close(b.d_density, a.d_density, 1e-12)
        assert np.allclose(b.d_group_w, a.d_group_w, rtol=1e-12, atol=0)
