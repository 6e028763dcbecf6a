"""Prescribed iteration counts: the sets that start no group are enqueued
without the group-start kernels, so the results equal those of a replayed chunk,
which keeps every launch, bit for bit; a source that turns non-finite ends the
solve with its error, and the solver stays usable."""
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


def _problem(scale=1.0, B=3):
    ph = I.abdomen_phantom(21, 18, 5, 38.4 / 21)
    xs = I.xs_tables(ph.material_names, 4, 1)
    dirs, w = I.lq_quadrature(4)
    pos, axis = I.ring_sources(B, 360.0 / B)
    return I.Problem("prescribed", ph, xs, dirs, w, 1, pos, axis, 20.0, 10.0, scale * I.kramers_weights(xs.edges))


@pytest.mark.parametrize("prec", ["fp32", "fp64", "fp32_bf16map"])
@pytest.mark.parametrize("fuse", [-1, 1])
def test_prescribed_equals_replay(fuse, prec):
    for fi in ([1, 1, 1, 1], [3, 1, 5, 2], [2, 9, 1, 1]):
        out = []
        for graph in (True, False):
            s = dctsn.Solver(_problem())
            try:
                st = s.solve(precision=prec, fuse_maps=fuse, use_graph=graph, fixed_iters=np.array(fi, dtype=np.int32))
                out.append((np.array(st.iters), s.dose(), s.moments(), np.array(st.balance)))
            finally:
                s.close()
        print(f"[prescribed] {prec} fuse {fuse} counts {fi}", flush=True)
        assert np.all(out[1][0] == np.array(fi))
        for a, b in zip(*out):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("fuse", [-1, 1])
def test_non_finite_source_ends(fuse):
    fi = np.array([3, 2, 2, 2], dtype=np.int32)
    s = dctsn.Solver(_problem(scale=1e60))     # beyond FP32
    try:
        with pytest.raises(dctsn.DctError) as e:
            s.solve(precision="fp32", fuse_maps=fuse, fixed_iters=fi)
        assert e.value.code == dctsn.DCT_ENUMERIC
        st = s.solve(precision="fp64", fuse_maps=fuse, fixed_iters=fi)
        assert np.all(np.array(st.iters) == fi) and np.all(np.isfinite(s.dose()))
    finally:
        s.close()
