"""The lattice sum's two series forms and the far fill's launch shapes.

  * g_p on the device against the oracle's Ewald sum for cells whose table
    holds monomials and for cells that keep Chebyshev series (tall structures,
    periods above the wavelength).  Tolerance: every term is fitted to 1e-14
    relative and 1e-15 absolute and terms below 1e-16 of g_p at the largest
    separation are dropped, which leaves a few 1e-13 of g_p: 1e-12 of
    max(|g_p|, 1 / (4 pi R_max)).
  * Z x of the symmetric fill against the plain one (another kernel, every
    ordered pair) with one and several test tetrahedra per wave and with
    ragged last blocks.  Tolerance: both round each entry a few times in
    1e-16, summed at random over N entries: 1e-13 relative to Z x.
"""
import numpy as np
import pytest

from oracle import pgf as OP
from paper_1809_05334_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vie():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1809_05334_amd import vie as V
    return V


@pytest.mark.parametrize("a,b,h,lam,th,ph", [
    (100.0, 100.0, 60.0, 600.0, 0.4, 0.3),      # monomials
    (157.0, 120.0, 110.0, 650.0, 0.0, 0.0),     # monomials, normal incidence
    (300.0, 240.0, 90.0, 400.0, 0.7, 0.3),      # several propagating orders
    (60.0, 60.0, 190.0, 550.0, 0.5, 0.2),       # Chebyshev: 3.2 periods tall
    (60.0, 60.0, 190.0, 550.0, 0.0, 0.0),
    (450.0, 450.0, 300.0, 330.0, 0.3, 0.5),     # Chebyshev: periods above the wavelength
])
def test_green_function_in_both_forms(vie, a, b, h, lam, th, ph):
    m = W.slab_mesh(a=a, b=b, thickness=h, nx=2, ny=2, nz=1)
    s = vie.Solver()
    s.upload_mesh(m)
    s.bind(vie.VIE_FP64, 10)
    s.fill(lam, th, ph, W.slab_eps(m))
    rng = np.random.default_rng(8)
    n = 300
    d = np.stack([rng.uniform(-a, a, n), rng.uniform(-b, b, n), rng.uniform(-h, h, n)], 1)
    d[:20, 2] = 0.0
    k = 2 * np.pi / lam
    kx, ky = k * np.sin(th) * np.cos(ph), k * np.sin(th) * np.sin(ph)
    # a sum that has converged on both sides for these cells
    ref = OP.pgf_ewald(d, k, kx, ky, a, b, M=7)
    got = s.pgf(d)
    floor = 1.0 / (4 * np.pi * np.sqrt(a * a + b * b + h * h))
    err = np.abs(got - ref) / np.maximum(np.abs(ref), floor)
    assert err.max() < 1e-12, err.max()
    s.close()


@pytest.mark.parametrize("nx,nz", [(2, 1), (3, 2), (5, 3), (8, 4), (9, 5)])
@pytest.mark.parametrize("theta", [0.0, 0.35])
def test_symmetric_and_plain_fills_agree_over_launch_shapes(vie, nx, nz, theta):
    m = W.slab_mesh(a=90.0, b=90.0, thickness=45.0, nx=nx, ny=nx, nz=nz)
    c = W.centroids(m.verts, m.tets)
    m.tet_domain = (c[:, 2] > 20.0).astype(np.int32)
    m.ndom = 2
    eps = np.where(m.tet_domain == 0, W.EPS_ACTIVE, W.EPS_SPACER)
    rng = np.random.default_rng(4)
    y = []
    for sym in (0, 1):
        s = vie.Solver()
        s.upload_mesh(m)
        s.set_option(vie.VIE_OPT_SYM_FILL, sym)
        s.bind(vie.VIE_FP64, 10)
        s.fill(600.0, theta, 0.4 if theta else 0.0, eps)
        assert s.fill_stats()["far_symmetric"] == sym
        N = s.num_unknowns()
        if not y:
            x = rng.standard_normal(N) + 1j * rng.standard_normal(N)
        y.append(s.apply_Z(x))
        s.close()
    assert np.linalg.norm(y[1] - y[0]) < 1e-13 * np.linalg.norm(y[0])
