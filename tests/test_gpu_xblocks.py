"""The fused map kernel on blocks of a row (rows too long for the LDS tile):
moments, dose and iteration counts equal the separate map kernels' bit for bit
over last blocks of one cell and more, blocks that the class rotation wraps
around, partial rows of y, prescribed and converged iteration counts."""
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


# nx, ny, nz, sources, S_N, P_N: P3 tiles of whole rows end at about 70 cells in
# FP64 and 145 in FP32
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,B,sn,L", [(129, 5, 2, 1, 6, 3), (83, 17, 3, 2, 6, 3), (96, 33, 1, 1, 8, 3),
                                             (200, 16, 2, 1, 6, 3), (177, 40, 1, 1, 8, 3), (161, 3, 1, 3, 6, 3)])
def test_blocks_match_separate_maps(nx, ny, nz, B, sn, L, prec):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, 2, L)
    dirs, w = I.lq_quadrature(sn)
    pos, axis = I.ring_sources(B, 360.0 / B)
    prob = I.Problem("xblocks", ph, xs, dirs, w, L, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))
    for kw in (dict(fixed_iters=np.array([3, 1], dtype=np.int32)), dict(tol=1e-4, max_iter=40)):
        out = []
        for fuse in (-1, 1):
            s = dctsn.Solver(prob)
            try:
                st = s.solve(precision=prec, fuse_maps=fuse, allow_notconv=True, **kw)
                out.append((np.array(st.iters), s.dose(), s.moments()))
            finally:
                s.close()
        print(f"[xblocks] {nx}x{ny}x{nz} B={B} S{sn} P{L} {prec} iters {out[0][0].ravel().tolist()}", flush=True)
        for a, b in zip(*out):
            assert np.array_equal(a, b)
