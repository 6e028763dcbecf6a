"""The fused map kernel on blocks of a row with more than 16 moments (P4, P5), on
blocks narrower than 64 cells and on rows barely longer than a block, so that the
class rotation wraps within it: moments and dose equal the separate map kernels'
bit for bit.  Block widths as the library chooses them: the fewest equal blocks
of at most 64 and at least 32 cells that fit the workgroup's LDS, else 32 and a rest."""
import numpy as np
import pytest

from paper_1811_12391_amd import dctsn, inputs as I

pytestmark = pytest.mark.gpu

LDS = 160 * 1024


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dctsn.lib()
    yield


def _product_quadrature(nmu, nphi):
    """Gauss-Legendre in z x equally spaced azimuths, octant by octant."""
    mu, wm = np.polynomial.legendre.leggauss(nmu)
    ph = (np.arange(nphi) + 0.5) * 2.0 * np.pi / nphi
    M, P = np.meshgrid(mu, ph, indexing="ij")
    s = np.sqrt(1.0 - M * M)
    d = np.stack([s * np.cos(P), s * np.sin(P), M], -1).reshape(-1, 3)
    w = np.repeat(wm, nphi) * 2.0 * np.pi / nphi
    o = np.lexsort((d[:, 0] < 0, d[:, 1] < 0, d[:, 2] < 0))
    d = d[o]
    return d / np.linalg.norm(d, axis=1, keepdims=True), w[o]


def _width(nx, N, L, size):
    """Cells of a block: nx when whole rows fit, 0 when no block does."""
    Nm = (L + 1) ** 2
    NmP, NcP = 16 * -(-Nm // 16), 16 * -(-(N // 2) // 16)

    def lds(xb):
        pitch = (xb | 1) + 1
        return size * (Nm * (16 * pitch + 4) + 2 * NmP * (NcP + 1) + 2 * NcP * (NmP + 1)) + 16 * N + 1024

    xb, n = nx, -(-nx // 64)
    while lds(xb) > LDS:
        xb, n = -(-nx // n), n + 1
        if xb < 32:
            return 32 if nx >= 32 and lds(32) <= LDS else 0
    return xb


# nx, ny, nz, L, precision, cells of a block
CASES = [(65, 19, 2, 4, "fp64", 33), (97, 16, 1, 4, "fp64", 33), (64, 5, 3, 4, "fp64", 32), (71, 5, 2, 4, "fp64", 32),
         (54, 18, 2, 4, "fp64", 32), (100, 33, 1, 4, "fp32", 50),
         (129, 17, 2, 5, "fp32", 43), (97, 3, 2, 5, "fp32", 49), (65, 50, 1, 5, "fp32", 33),
         (68, 33, 2, 3, "fp64", 34), (131, 9, 2, 2, "fp64", 44), (77, 20, 1, 3, "fp64", 39)]


@pytest.mark.parametrize("nx,ny,nz,L,prec,xb", CASES)
def test_narrow_blocks_match_separate_maps(nx, ny, nz, L, prec, xb):
    ph = I.abdomen_phantom(nx, ny, nz, 38.4 / max(nx, ny))
    xs = I.xs_tables(ph.material_names, 2, L)
    dirs, w = _product_quadrature(6, 12) if L > 3 else I.lq_quadrature(8)
    assert _width(nx, len(w), L, 8 if prec == "fp64" else 4) == xb < nx
    pos, axis = I.ring_sources(2, 180.0)
    prob = I.Problem("orders", ph, xs, dirs, w, L, pos, axis, 20.0, 10.0, I.kramers_weights(xs.edges))
    for kw in (dict(fixed_iters=np.array([3, 1], dtype=np.int32)), dict(tol=1e-4, max_iter=40)):
        out = []
        for fuse in (-1, 1):
            s = dctsn.Solver(prob)
            try:
                st = s.solve(precision=prec, fuse_maps=fuse, allow_notconv=True, **kw)
                assert st.fused_maps == (fuse == 1)
                out.append((np.array(st.iters), s.dose(), s.moments()))
            finally:
                s.close()
        print(f"[orders] {nx}x{ny}x{nz} P{L} {prec} blocks of {xb}", flush=True)
        for a, b in zip(*out):
            assert np.array_equal(a, b)
