"""Group transitions on both splits of the grid (256 consecutive voxels, 16 x 16
patches of a layer): thin grids whose patches would be mostly empty, grids with
partial patches, with separate maps (the transition lays the first source out)
and fused ones (it does not), cold and warm, against the oracle."""
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


@pytest.mark.parametrize("nx,ny,nz,B", [(1, 1, 300, 1), (300, 1, 2, 2), (2, 290, 3, 1), (17, 33, 3, 2), (16, 16, 2, 1),
                                        (40, 9, 5, 3)])
def test_transitions_match_oracle(nx, ny, nz, B):
    import oracle

    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny, 64))
    xs = I.xs_tables(ph.material_names, 3, 1)
    dirs, w = I.lq_quadrature(4)
    pos, axis = I.ring_sources(B, 360.0 / B)
    prob = I.Problem("transition", ph, xs, dirs, w, 1, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))
    fi = np.array([3, 1, 2], dtype=np.int32)
    ref = oracle.solve_problem(prob, fixed_iters=fi)
    for fuse in (-1, 1):
        s = dctsn.Solver(prob)
        try:
            for kw in (dict(), dict(chunk=1), dict(use_graph=True)):
                st = s.solve(precision="fp64", fixed_iters=fi, fuse_maps=fuse, **kw)
                d = s.dose()
                print(f"[transition] {nx}x{ny}x{nz} B={B} fuse {fuse} {kw} fused {st.fused_maps}", flush=True)
                assert np.abs(d - ref.dose).max() <= 1e-10 * np.abs(ref.dose).max()
                assert np.allclose(st.balance[..., 0], np.asarray(ref.balance)[..., 0], rtol=1e-10, atol=1e-300)
            cold = s.moments()
            # a warm solve converges to the cold one's fixed point and closes its balance
            s.solve(precision="fp64", tol=1e-12, fuse_maps=fuse)
            m0 = s.moments()
            st = s.solve(precision="fp64", tol=1e-12, fuse_maps=fuse, warm_start=True)
            assert st.warm_start == 1
            assert np.abs(s.moments() - m0).max() <= 1e-9 * np.abs(m0).max()
            P, R, Lk = np.moveaxis(st.balance, -1, 0)
            assert np.max(np.abs(P - R - Lk) / P) < 1e-9
            assert cold.shape == m0.shape
        finally:
            s.close()
