"""Sweeps of waves of 64 rows (couplings 1 - 3) on grids whose 16-row pieces keep
to 64-byte boundaries and on grids where they straddle them, one block and
several: every coupling's dose and moments are the tile waves' (coupling 4, or
the untuned choice of taller grids) bit for bit."""
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


def _run(prob, **kw):
    s = dctsn.Solver(prob)
    try:
        st = s.solve(fixed_iters=np.full(prob.G, 3, dtype=np.int32), **kw)
        return st, s.dose(), s.moments()
    finally:
        s.close()


# rows of 16, 8 and an odd remainder; 11 and 12 layers are workgroups of which
# two share a compute unit, 13 of which one does
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,B", [(20, 16, 11, 3), (21, 24, 12, 1), (19, 37, 13, 2), (24, 80, 33, 1),
                                        (33, 72, 18, 1), (33, 71, 18, 2)])
def test_couplings_bitwise(nx, ny, nz, B, prec):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, 2, 1)
    dirs, w = I.lq_quadrature(4)
    pos, axis = I.ring_sources(B, 360.0 / B)
    prob = I.Problem("rows", ph, xs, dirs, w, 1, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))
    one = ny <= 64 and nz <= 16
    st, d, m = _run(prob, precision=prec, **(dict(sweep_bk=16, sweep_sync=4) if one else {}))
    assert st.sweep_sync == 4
    for bk, sync in ((16, 1), (16, 2), (4, 1), (4, 2), (4, 3)):
        print(f"[rows] {nx}x{ny}x{nz} B={B} {prec} {bk}:{sync}", flush=True)
        st2, d2, m2 = _run(prob, precision=prec, sweep_bk=bk, sweep_sync=sync)
        assert st2.sweep_sync == sync
        assert np.array_equal(d2, d) and np.array_equal(m2, m)
