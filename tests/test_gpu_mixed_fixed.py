"""The mixed-precision operator's FP32 entries to the bit, and its solution.

Every far contribution is added to its FP32 entry and rounded, so a fill whose
FP64 arithmetic moves by a rounding moves isolated entries to the neighbouring
FP32 value (1e-7 of them) and a component of the solution by up to 1e-7.  The
far entries are therefore held to the bit, by digests of cells with an uneven
mesh (N = 3,038), with the symmetric and the plain fill, at oblique and normal
incidence, alone and in a batch.  Entries of touching elements hold FP64 parts
and are left out.

The solution against the FP64 operator's: an entry is the sum of at most four
contributions and one transposed block, each rounded once, 5 * 2^-24 = 3e-7
relative to the largest of them; a condition of Z below 1e2 for these cells
gives 3e-5 in norm, and ten times that for the worst component (relative to
the larger of it and the vector's root mean square)."""
import hashlib

import numpy as np
import pytest

from oracle import topology as OT
from paper_1809_05334_amd import workloads as W

pytestmark = pytest.mark.gpu

CELL = (157.0, 71.0, 43.0, 17.0, 15.6, 39.0)
DIGESTS = {   # (symmetric fill, theta)
    (1, 0.5): "4ec728f0f9b6a59dabf124c01510eaaa",
    (1, 0.0): "010a1e427af1ba05d90885e1e2c2ee88",
    (0, 0.5): "3b42c8967933640354bb104a4d797ce4",
    (0, 0.0): "8a2eda86dde73fffb4de13f69a9c0305",
}
TALL_DIGEST = "19699c42b6007eb41a3fb7afba67da5a"


@pytest.fixture(scope="module")
def vie():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1809_05334_amd import vie as V
    return V


@pytest.fixture(scope="module")
def cell():
    m = W.osc_cell_mesh(*CELL)
    t = OT.build(m.verts, m.tets, m.tet_domain, m.ndom, m.a, m.b)
    return m, far_mask(t)


def far_mask(t):
    """[N, N]: no tetrahedron of the row's unknown shares a vertex with one of the column's."""
    N = len(t.tplus)
    at = np.zeros((N, t.ncanon), np.float32)   # vertices of an unknown's tetrahedra
    for half in (t.tplus, t.tminus):
        ok = np.nonzero(half >= 0)[0]
        at[np.repeat(ok, 4), t.canon[t.tets[half[ok]]].ravel()] = 1
    return at @ at.T == 0


def make(vie, m, sym, precision=None):
    s = vie.Solver()
    s.upload_mesh(m)
    s.set_option(vie.VIE_OPT_SYM_FILL, sym)
    s.bind(vie.VIE_MIXED_FP32 if precision is None else precision, 100)
    return s


def digest(s, far):
    rows, cols = np.nonzero(far)
    h = hashlib.sha256()
    for lo in range(0, len(rows), 1 << 21):
        z = s.read_Z(rows[lo:lo + (1 << 21)], cols[lo:lo + (1 << 21)])
        f = z.astype(np.complex64)
        assert np.array_equal(f.astype(np.complex128), z)   # FP32 values, no near part
        h.update(np.ascontiguousarray(f).tobytes())
    return h.hexdigest()[:32]


@pytest.mark.parametrize("sym,theta", list(DIGESTS))
def test_far_entries_are_the_recorded_ones(vie, cell, sym, theta):
    m, far = cell
    s = make(vie, m, sym)
    s.fill(612.0, theta, 0.7, W.osc_eps(m, 612.0))
    assert digest(s, far) == DIGESTS[sym, theta]
    s.close()


def tall_slab():
    """A slab of four periods' height above the wavelength (N = 1,952), whose
    lattice sum has more terms than an oblique symmetric fill takes."""
    m = W.slab_mesh(500.0, 400.0, 1700.0, 4, 4, 10)
    t = OT.build(m.verts, m.tets, m.tet_domain, m.ndom, m.a, m.b)
    return m, far_mask(t)


def test_a_tall_cell_at_oblique_incidence_takes_the_plain_fill(vie):
    m, far = tall_slab()
    s = make(vie, m, 1)
    s.fill(360.0, 0.4, 0.3, W.slab_eps(m))
    assert s.fill_stats()["far_symmetric"] == 0
    assert digest(s, far) == TALL_DIGEST
    s.close()


@pytest.mark.parametrize("sym", [0, 1])
def test_far_entries_in_a_batch(vie, cell, sym):
    import torch
    m, far = cell
    stream = torch.cuda.Stream()
    small = W.slab_mesh(nx=3, ny=3, nz=2)
    cells = [small, m, m]
    solvers = []
    for c in cells:
        s = vie.Solver(0, stream=stream)
        s.upload_mesh(c)
        s.set_option(vie.VIE_OPT_SYM_FILL, sym)
        s.bind(vie.VIE_MIXED_FP32, 100)
        solvers.append(s)
    b = vie.Batch(solvers, stream=stream)
    b.fill([600.0, 612.0, 612.0], [0.3, 0.5, 0.0], [0.2, 0.7, 0.7],
           [W.slab_eps(small), W.osc_eps(m, 612.0), W.osc_eps(m, 612.0)])
    assert digest(solvers[1], far) == DIGESTS[sym, 0.5]
    assert digest(solvers[2], far) == DIGESTS[sym, 0.0]
    b.close()
    for s in solvers:
        s.close()


@pytest.mark.parametrize("cell_args", [(200.0, 80.0, 40.0, 20.0, 8.7, 20.0), (200.0, 80.0, 40.0, 20.0, 5.0, 20.0)],
                         ids=["N18590", "N37376"])
def test_solution_against_the_fp64_operators(vie, cell_args):
    m = W.osc_cell_mesh(*cell_args)
    eps = W.osc_eps(m, 640.0)
    x = []
    for precision in (vie.VIE_FP64, vie.VIE_MIXED_FP32):
        s = make(vie, m, 1, precision)
        s.fill(640.0, 0.6, 0.4, eps)
        s.factor()
        s.solve_pair()
        x.append([s.read_solution(pol) for pol in (vie.VIE_TE, vie.VIE_TM)])
        s.close()
    for ref, got in zip(*x):
        rms = np.linalg.norm(ref) / np.sqrt(ref.size)
        assert np.linalg.norm(got - ref) < 3e-5 * np.linalg.norm(ref)
        assert np.max(np.abs(got - ref) / np.maximum(rms, np.abs(ref))) < 3e-4
