"""Read-out of the dose and fluences over the numbers of right-hand sides and
groups where its work split changes: fewer and more right-hand sides than a
workgroup has waves, groups that are no multiple of the loads in flight, grids
that end inside a wave.  The dose is sum_g kappa_g (phi_u,g + phi_c,g) in group
order, the summed dose the per-source doses added in their order."""
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


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,B,S,G", [(1, 1, 1, 1, 1, 1), (5, 7, 3, 1, 1, 5), (13, 5, 2, 7, 1, 4),
                                            (8, 8, 1, 8, 1, 3), (11, 9, 4, 18, 2, 6), (7, 9, 2, 17, 1, 9)])
def test_readout(nx, ny, nz, B, S, G, prec):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, G, 1)
    dirs, w = I.lq_quadrature(4)
    pos, axis = I.ring_sources(B, 360.0 / B)
    prob = I.Problem("readout", ph, xs, dirs, w, 1, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))
    s = dctsn.Solver(prob)
    try:
        s.solve(precision=prec, fixed_iters=np.full(G, 2, dtype=np.int32), superpose=S)
        dose, pu, pc = s.dose(want_phi=True)
        tot = s.dose(summed=True)
    finally:
        s.close()
    print(f"[readout] {nx}x{ny}x{nz} B={B} S={S} G={G} {prec}", flush=True)
    kap = np.asarray(xs.kerma)[ph.material]                       # [C][G]
    want = np.einsum("cg,bgc->bc", kap, pu + pc)
    # G rounded products and sums of non-negative terms
    assert np.all(np.abs(dose - want) <= (G + 2) * 2.0 ** -52 * np.abs(want))
    seq = np.zeros(ph.C)
    for b in range(B // S):
        seq = seq + dose[b]
    assert np.array_equal(tot, seq)
