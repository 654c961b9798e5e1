"""The Arnoldi step's tiles: basis counts at and around the 64 vectors that an
update takes at a time and the 128 rotations of a Givens pass, and more rows
than the update's blocks hold at once.  In exact arithmetic the residual
estimate of a restart cycle is the true residual at its end; in FP64 CGS2 keeps
the basis orthogonal to rounding, so the two differ by some 1e-16 times the
condition of Z M^-1 relative to b: 1e-9 absolute here."""
import numpy as np
import pytest

from gpu_cases import eps_for, osc_small
from paper_1809_05334_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vie():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1809_05334_amd import vie as V
    return V


@pytest.mark.parametrize("steps", [1, 2, 63, 64, 65, 127, 128, 129, 200])
def test_estimate_equals_true_residual_after_one_cycle(vie, steps):
    m = osc_small()
    s = vie.Solver()
    s.upload_mesh(m)
    s.bind(vie.VIE_FP64, 200)
    s.set_option(vie.VIE_OPT_PRECOND, 1)
    s.fill(480.0, 0.3, 0.2, eps_for(m, 480.0))
    info = s.solve(1, tol=1e-14, max_iter=steps, restart=steps, allow_noconv=True)
    h = s.residual_history()
    # every step is taken unless the estimate meets the tolerance before that
    assert info["iters"] == len(h) and (len(h) == steps or h[-1] <= 1e-14)
    assert np.all(np.diff(h) <= 1e-12)
    assert abs(info["true_rel_residual"] - h[-1]) < 1e-9
    s.close()


def test_estimate_equals_true_residual_on_many_rows(vie):
    xs, zs = np.linspace(0.0, 120.0, 25), np.linspace(0.0, 100.0, 21)
    verts, tets = W.brick_grid_mesh(xs, xs, zs)
    m = W.Mesh(verts, tets, np.zeros(len(tets), np.int32), 1, 120.0, 120.0, (xs, xs, zs))
    s = vie.Solver()
    s.upload_mesh(m)
    s.bind(vie.VIE_GRID_FP64, 6)
    assert s.num_unknowns() > 512 * 256
    s.set_option(vie.VIE_OPT_PRECOND, 1)
    s.fill(600.0, 0.3, 0.2, W.slab_eps(m))
    info = s.solve(1, tol=1e-14, max_iter=6, restart=6, allow_noconv=True)
    h = s.residual_history()
    assert abs(info["true_rel_residual"] - h[-1]) < 1e-9
    s.close()
