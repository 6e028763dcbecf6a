"""Sweeps whose workgroups wait for each other (tile waves in z groups, chosen
untuned): when such a wait gives up, the call runs again without them and later
calls on the context avoid them; couplings asked for by number still fail, and
the next call finds its hand-over buffers empty.  The failure is a flag set by
the host (dct_test_fail_waits); nothing goes wrong on the device."""
import ctypes as ct

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


def _fail_waits(solver, n=1):
    f = dctsn.lib().dct_test_fail_waits
    f.argtypes, f.restype = [ct.c_void_p, ct.c_int], ct.c_int
    assert f(solver.h, n) == dctsn.DCT_OK


def _problem(nx=33, ny=70, nz=18):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, 2, 1)
    dirs, w = I.lq_quadrature(4)
    pos, axis = I.ring_sources(1, 360.0)
    return I.Problem("fallback", ph, xs, dirs, w, 1, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))


FI = np.array([3, 2], dtype=np.int32)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_solve_runs_again_without_waits(prec):
    prob = _problem()
    s = dctsn.Solver(prob)
    try:
        a = s.solve(precision=prec, fixed_iters=FI)
        d, m = s.dose(), s.moments()
        assert a.sweep_sync == 4
        for kw in (dict(), dict(chunk=1), dict(use_graph=True)):
            _fail_waits(s)
            b = s.solve(precision=prec, fixed_iters=FI, **kw)
            assert np.array_equal(s.dose(), d) and np.array_equal(s.moments(), m)
            assert np.array_equal(b.iters, a.iters) and b.status == dctsn.DCT_OK
            _fail_waits(s, 0)
            c = s.solve(precision=prec, fixed_iters=FI, **kw)
            assert np.array_equal(s.dose(), d) and np.array_equal(c.eps, a.eps)
            s.close()
            s = dctsn.Solver(prob)
    finally:
        s.close()


def test_second_failure_is_reported():
    """With no waits between workgroups left to avoid, the flag is an error."""
    s = dctsn.Solver(_problem())
    try:
        _fail_waits(s, 2)
        with pytest.raises(dctsn.DctError) as e:
            s.solve(precision="fp64", fixed_iters=FI)
        assert e.value.code == dctsn.DCT_EDEVICE
        s.solve(precision="fp64", fixed_iters=FI)
    finally:
        s.close()


def test_adjoint_runs_again_without_waits():
    prob = _problem()
    roi = np.random.default_rng(5).random(prob.phantom.C)
    s = dctsn.Solver(prob)
    try:
        assert s.solve(precision="fp64", fixed_iters=FI, keep_adjoint=True).sweep_sync == 4
        a = s.adjoint(roi, fixed_iters=FI)
        _fail_waits(s)
        b = s.adjoint(roi, fixed_iters=FI)
        c = s.adjoint(roi, fixed_iters=FI)
    finally:
        s.close()
    for x in (b, c):
        assert x.R == a.R and np.array_equal(x.eps, a.eps)
        assert np.allclose(x.d_density, a.d_density, rtol=0, atol=1e-12 * np.abs(a.d_density).max())
        assert np.allclose(x.d_group_w, a.d_group_w, rtol=1e-12, atol=0)


def test_pipelined_blocks_fail_and_recover():
    """Coupling 3 was asked for: the call fails, and the next solve and adjoint
    start from empty faces."""
    prob = _problem()
    roi = np.random.default_rng(5).random(prob.phantom.C)
    kw = dict(precision="fp64", fixed_iters=FI, keep_adjoint=True, sweep_bk=6, sweep_sync=3)
    s = dctsn.Solver(prob)
    try:
        assert s.solve(**kw).sweep_sync == 3
        d, a = s.dose(), s.adjoint(roi, fixed_iters=FI)
        _fail_waits(s)
        with pytest.raises(dctsn.DctError):
            s.adjoint(roi, fixed_iters=FI)
        b = s.adjoint(roi, fixed_iters=FI)
        _fail_waits(s)
        with pytest.raises(dctsn.DctError):
            s.solve(**kw)
        s.solve(**kw)
        assert np.array_equal(s.dose(), d)
    finally:
        s.close()
    assert np.allclose(b.d_density, a.d_density, rtol=0, atol=1e-12 * np.abs(a.d_density).max())


def test_failed_solve_leaves_no_warm_start():
    """A failed solve has overwritten the moments: the next warm solve starts
    from zero; a warm solve that runs again does too."""
    prob = _problem()
    s = dctsn.Solver(prob)
    try:
        kw = dict(precision="fp64", tol=1e-10, sweep_bk=16, sweep_sync=2)
        ref = s.solve(**kw)
        assert s.solve(warm_start=True, **kw).warm_start == 1
        _fail_waits(s)
        with pytest.raises(dctsn.DctError):
            s.solve(**kw)
        st = s.solve(warm_start=True, **kw)
        assert st.warm_start == 0 and np.array_equal(st.iters, ref.iters)
        _fail_waits(s)
        st = s.solve(precision="fp64", tol=1e-10, warm_start=True)
        assert st.warm_start == 0 and np.array_equal(st.iters, ref.iters)
    finally:
        s.close()
    s = dctsn.Solver(prob)
    try:
        # prescribed counts from moments that are gone cannot be repeated
        s.solve(precision="fp64", fixed_iters=FI)
        _fail_waits(s)
        with pytest.raises(dctsn.DctError) as e:
            s.solve(precision="fp64", fixed_iters=FI, warm_start=True)
        assert e.value.code == dctsn.DCT_EDEVICE
    finally:
        s.close()


def test_pipelined_blocks_on_a_buffer_of_another_shape():
    """The hand-over buffers are as large as the largest solve so far: a small
    pipelined solve and then a large one find them empty throughout."""
    big, small = _problem(40, 130, 20), _problem(12, 70, 4)
    kw = dict(precision="fp64", fixed_iters=FI, sweep_bk=4, sweep_sync=3)
    def load(s, prob):
        ph, xs = prob.phantom, prob.xs
        dctsn.set_geometry(s.h, ph.nx, ph.ny, ph.nz, ph.dx, ph.dy, ph.dz, ph.origin, ph.material, ph.density)
        dctsn.set_xs(s.h, xs.G, xs.edges, xs.M, prob.L, xs.sigma_t, xs.sigma_s[:, : prob.L + 1], xs.kerma)
        dctsn.set_source(s.h, prob.B, prob.src_pos, prob.src_axis, prob.fan_deg, prob.cone_deg, prob.group_w)
        s.prob = prob

    s = dctsn.Solver(big)
    try:
        s.solve(precision="fp64", fixed_iters=FI, sweep_bk=16, sweep_sync=2)
        d = s.dose()
        load(s, small)
        assert s.solve(**dict(kw, sweep_bk=2)).sweep_sync == 3
        load(s, big)
        assert s.solve(**kw).sweep_sync == 3
        assert np.array_equal(s.dose(), d)
    finally:
        s.close()
