"""Timed work of the library: what a program that models plasmonic cells asks of it.

A case is one of these kinds of work, at a size, a storage precision and the
options that such a program sets:

  request   everything for one incidence: fill, factor, solve, absorptance, R and T
            (optionally the absorption per tetrahedron and the field on a plane)
  fill      a new wavelength or angle on a resident mesh, then one product Z x
  factor    the block factors of a filled matrix, applied to one vector
  pair      TE and TM solved on a filled and factored matrix
  batch     several uneven cells filled, factored and solved together
  grid      the structured-grid operator: a fill and a product, or a product alone
  pgf       samples of the periodic Green's function

Cells are the plasmonic cell (layers and a metal sphere) and the homogeneous
slab of paper_1809_05334_amd.workloads.  The seed of a case gives what changes
from call to call in a sweep or a request stream: wavelength, angles,
permittivities of the layers and the vectors of products.  Solves use the
entry points' default tolerance, 1e-12.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1809_05334_amd import vie
from paper_1809_05334_amd import workloads as W

PRECISION = {"fp64": vie.VIE_FP64, "mixed": vie.VIE_MIXED_FP32, "grid": vie.VIE_GRID_FP64}
RESTART = 100
# Krylov steps that every solve of these cells takes at the least (42 and more were seen at 1e-8)
ITERS = 40


# ------------------------------------------------------------------ the cases
def _osc(a, t_active, t_spacer, radius, h_fine, h_coarse):
    return {"shape": "osc", "a": a, "t_active": t_active, "t_spacer": t_spacer, "radius": radius, "h_fine": h_fine,
            "h_coarse": h_coarse}


def _slab(a, thickness, nx, nz):
    return {"shape": "slab", "a": a, "thickness": thickness, "nx": nx, "nz": nz}


def listed():
    bench = (200.0, 80.0, 40.0, 20.0)   # the plasmonic cell of the benchmark: period, layers, sphere radius
    return [
        # the smallest call: the 100 nm slab (N = 416) of the parity tests, one polarisation; launches and host work
        {"name": "request_slab_fp64", "kind": "request", "precision": "fp64", "sym": 0, "oblique": 1, "pair": 0,
         "maps": 0, **_slab(100.0, 50.0, 4, 2)},
        # an ordinary request of the serving trace (N = 3,038), one polarisation, symmetric fill as the server sets it
        {"name": "request_small_mixed", "kind": "request", "precision": "mixed", "sym": 1, "oblique": 1, "pair": 0,
         "maps": 0, **_osc(157.0, 71.0, 43.0, 17.0, 15.6, 39.0)},
        # one incidence of a study with maps: FP64, default options, both polarisations, normal incidence (N = 6,272)
        {"name": "request_maps_fp64", "kind": "request", "precision": "fp64", "sym": 0, "oblique": 0, "pair": 1,
         "maps": 1, **_osc(120.0, 80.0, 40.0, 20.0, 10.0, 24.0)},
        # one incidence of the angular sweep on the mixed path, both polarisations, at the benchmark cell's 5 nm mesh (N = 37,376)
        {"name": "sweep_large_mixed", "kind": "request", "precision": "mixed", "sym": 1, "oblique": 1, "pair": 1,
         "maps": 0, **_osc(*bench, 5.0, 20.0)},
        # a new angle on a resident FP64 matrix, default options (every ordered pair; N = 18,590)
        {"name": "fill_fp64", "kind": "fill", "precision": "fp64", "sym": 0, "oblique": 1,
         **_osc(200.0, 80.0, 40.0, 20.0, 8.7, 20.0)},
        # a new angle on the largest matrix of these cases, mixed path with the symmetric fill (N = 37,376)
        {"name": "fill_large_mixed", "kind": "fill", "precision": "mixed", "sym": 1, "oblique": 1, **_osc(*bench, 5.0, 20.0)},
        # FP64 block factors of a middle-sized cell (N = 15,840), applied once
        {"name": "factor_fp64", "kind": "factor", "precision": "fp64", "sym": 1, "oblique": 1,
         **_osc(200.0, 80.0, 40.0, 20.0, 7.3, 30.0)},
        # another incidence's Krylov solve in FP64: products and triangular solves for two vectors
        {"name": "pair_fp64", "kind": "pair", "precision": "fp64", "sym": 1, "oblique": 1,
         **_osc(200.0, 80.0, 40.0, 20.0, 7.3, 30.0)},
        # a wave of six uneven cells of the batched workload on the mixed path
        {"name": "batch_mixed", "kind": "batch", "precision": "mixed", "sym": 1, "cells": 6, "cell_seed": 5,
         "n_lo": 2000, "n_hi": 9000},
        # the structured-grid operator on a small uniform cell (N = 9,344): fill and product
        {"name": "grid_fill", "kind": "grid", "product_only": 0, "oblique": 1, **_osc(80.0, 80.0, 40.0, 20.0, 10.0, 10.0)},
        # its product on the uniform 5 nm grid of the benchmark stack (N = 74,240): one Krylov step's operator
        {"name": "grid_product_large", "kind": "grid", "product_only": 1, "oblique": 1,
         **_osc(80.0, 80.0, 40.0, 20.0, 5.0, 5.0)},
        # Green's function samples over a cell
        {"name": "pgf_samples", "kind": "pgf", "points": 20011, "oblique": 1, **_slab(200.0, 120.0, 4, 3)},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_osc(rng, n_lo, n_hi):
    """A cell of the batched workload's ranges whose unknowns come out near a target drawn in [n_lo, n_hi]."""
    target = _log(rng, n_lo, n_hi)
    a, t_act, t_sp = rng.uniform(100.0, 300.0), rng.uniform(60.0, 100.0), rng.uniform(30.0, 60.0)
    radius = rng.uniform(10.0, min(40.0, t_sp / 2))
    h_c = rng.uniform(20.0, min(40.0, a / 3.0))
    h_f = 3.0
    while h_f < h_c and _count(a, t_act, t_sp, radius, h_f, h_c) > target:
        h_f *= 1.03
    return _osc(round(a, 1), round(t_act, 1), round(t_sp, 1), round(radius, 1), round(h_f, 2), round(h_c, 1))


def _count(a, t_act, t_sp, radius, h_f, h_c):
    xs = W.graded_axis(a, a / 2 - radius, a / 2 + radius, h_f, h_c)
    zs = np.concatenate([W.graded_axis(t_act, 0, 0, h_f, h_c), t_act + W.graded_axis(t_sp, 0, t_sp, h_f, h_c)[1:]])
    return W.count_unknowns_paired(xs, xs, zs)


def draw(rng):
    kind = rng.choice(["request", "request", "fill", "fill", "factor", "pair", "batch", "grid", "pgf"])
    precision, sym, oblique = rng.choice(["fp64", "mixed"]), rng.randint(0, 1), int(rng.random() < 0.75)
    if kind == "request":
        cell = _draw_osc(rng, 1500, 25000)
        if rng.random() < 0.25:
            nx = rng.randint(2, 8)
            cell = _slab(round(rng.uniform(60.0, 200.0), 1), round(rng.uniform(30.0, 100.0), 1), nx, rng.randint(1, 4))
        return {"kind": kind, "precision": precision, "sym": sym, "oblique": oblique, "pair": rng.randint(0, 1),
                "maps": int(rng.random() < 0.3), **cell}
    if kind == "fill":
        return {"kind": kind, "precision": precision, "sym": sym, "oblique": oblique, **_draw_osc(rng, 1500, 30000)}
    if kind == "factor":   # FP64: the factors themselves come back, through one apply
        return {"kind": kind, "precision": "fp64", "sym": 1, "oblique": oblique, **_draw_osc(rng, 1500, 18000)}
    if kind == "pair":
        return {"kind": kind, "precision": precision, "sym": 1, "oblique": oblique, **_draw_osc(rng, 1500, 18000)}
    if kind == "batch":
        return {"kind": kind, "precision": precision, "sym": sym, "cells": rng.randint(2, 6),
                "cell_seed": rng.randint(0, 10 ** 6), "n_lo": 2000, "n_hi": 9000}
    if kind == "grid":
        # uniform bricks: the sphere's span has to start and end on grid planes
        h = rng.choice([12.0, 10.0, 8.0, 5.0])
        n, n_act, n_sp = rng.randint(3, int(80 / h)), rng.randint(2, int(80 / h)), rng.randint(1, int(40 / h))
        radius = h * (0.5 if n % 2 else 1.0)
        return {"kind": kind, "product_only": rng.randint(0, 1), "oblique": oblique,
                **_osc(h * n, h * n_act, h * n_sp, radius, h, h)}
    return {"kind": kind, "points": int(_log(rng, 100, 60000)), "oblique": oblique,
            **_slab(round(rng.uniform(60.0, 300.0), 1), round(rng.uniform(30.0, 200.0), 1), 4, 3)}


# ------------------------------------------------------------------ inputs
def _mesh(case):
    if case["shape"] == "slab":
        return W.slab_mesh(case["a"], case["a"], case["thickness"], case["nx"], case["nx"], case["nz"])
    return W.osc_cell_mesh(case["a"], case["t_active"], case["t_spacer"], case["radius"], case["h_fine"], case["h_coarse"])


def _wave(case, rng):
    """Wavelength and incidence of one call, clear of the Rayleigh-Wood anomalies (the library refuses those)."""
    a = case["a"]
    while True:
        lam = rng.uniform(500.0, 800.0)
        theta = math.radians(rng.uniform(5.0, 60.0)) if case["oblique"] else 0.0
        phi = math.radians(rng.uniform(0.0, 90.0)) if case["oblique"] else 0.0
        if W.wood_margin(a, a, lam, theta, phi) > 0.05:
            return lam, theta, phi


def _eps(case, mesh, lam, rng):
    """Permittivity per tetrahedron: the stand-in constants, a few per cent apart from call to call."""
    if case["shape"] == "slab":
        return W.slab_eps(mesh, W.EPS_SLAB * rng.uniform(0.95, 1.05))
    return W.osc_eps(mesh, lam, W.EPS_ACTIVE * rng.uniform(0.95, 1.05), W.EPS_SPACER * rng.uniform(0.95, 1.05))


def _bound(mesh, precision, sym):
    s = vie.Solver(0)
    s.upload_mesh(mesh)
    if sym:
        s.set_option(vie.VIE_OPT_SYM_FILL, 1)
    s.bind(precision, RESTART)
    return s


def _vector(rng, n):
    return rng.standard_normal(n) + 1j * rng.standard_normal(n)


def _separations(case, rng):
    """Separations inside the cell, none closer to a lattice point than 1 nm."""
    a, h, n = case["a"], case["thickness"], case["points"]
    d = np.stack([rng.uniform(-a, a, n), rng.uniform(-a, a, n), rng.uniform(-h, h, n)], 1)
    near = np.hypot(np.hypot(d[:, 0] - a * np.rint(d[:, 0] / a), d[:, 1] - a * np.rint(d[:, 1] / a)), d[:, 2]) < 1.0
    d[near, 2] = h / 2
    return d


def prepare(case, seed):
    rng = np.random.default_rng([seed, 77])
    if case["kind"] == "batch":
        return _prepare_batch(case, rng)
    mesh = _mesh(case)
    lam, theta, phi = _wave(case, rng)
    state = {"case": case, "wave": (lam, theta, phi), "eps": _eps(case, mesh, lam, rng)}
    kind = case["kind"]
    if kind == "grid":
        s = _bound(mesh, vie.VIE_GRID_FP64, 0)
    elif kind == "pgf":
        s = _bound(mesh, vie.VIE_FP64, 0)
    else:
        s = _bound(mesh, PRECISION[case["precision"]], case["sym"])
    state["solver"] = s
    if kind == "request":
        state["pol"] = vie.VIE_TM if case["oblique"] else vie.VIE_TE
        if case["maps"]:   # a plane through the middle of the cell, off the mesh planes
            top = mesh.grid[2][-1]
            x, z = np.meshgrid((np.arange(64) + 0.5) * case["a"] / 64, (np.arange(48) + 0.5) * top / 48, indexing="ij")
            state["points"] = np.stack([x.ravel(), np.full(x.size, case["a"] / 2 + 0.37), z.ravel()], 1)
    elif kind == "pgf":
        s.fill(lam, theta, phi, state["eps"])
        state["delta"] = _separations(case, rng)
    else:
        state["x"] = _vector(rng, s.num_unknowns())
        if kind in ("factor", "pair") or case.get("product_only"):
            s.fill(lam, theta, phi, state["eps"])
        if kind == "pair":
            s.factor()
    return state


def _prepare_batch(case, rng):
    cells = W.batch_cells(case["cells"], seed=case["cell_seed"], n_lo=case["n_lo"], n_hi=case["n_hi"])
    stream = torch.cuda.Stream()
    solvers, waves, eps = [], [], []
    for c in cells:
        mesh = W.cell_mesh(c)
        s = vie.Solver(0, stream=stream)
        s.upload_mesh(mesh)
        if case["sym"]:
            s.set_option(vie.VIE_OPT_SYM_FILL, 1)
        s.bind(PRECISION[case["precision"]], RESTART)
        lam, theta, phi = _wave({"a": c["a"], "oblique": 1}, rng)
        solvers.append(s)
        waves.append((lam, theta, phi))
        eps.append(_eps({"shape": "osc"}, mesh, lam, rng))
    return {"case": case, "batch": vie.Batch(solvers, stream=stream), "solvers": solvers, "waves": waves, "eps": eps,
            "pols": [c["pol"] for c in cells]}


# ------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        b = state["batch"]
        lams, thetas, phis = zip(*state["waves"])
        b.fill(lams, thetas, phis, state["eps"])
        b.factor()
        b.solve(state["pols"], tol=1e-12, restart=RESTART)
        return [{"x": s.read_solution(), "ART": s.absorption()} for s in state["solvers"]]
    s = state["solver"]
    if kind == "pgf":
        return s.pgf(state["delta"])
    if kind == "factor":
        s.factor()
        return s.precond_apply(state["x"])
    if kind == "pair":
        s.solve_pair()
        return [s.read_solution(pol) for pol in (vie.VIE_TE, vie.VIE_TM)]
    if not case.get("product_only"):
        s.fill(*state["wave"], state["eps"])
    if kind in ("fill", "grid"):
        return s.apply_Z(state["x"])
    s.factor()
    if case["pair"]:
        s.solve_pair()
        pols = [vie.VIE_TE, vie.VIE_TM]
    else:
        s.solve(state["pol"])
        pols = [state["pol"]]
    out = []
    for pol in pols:
        got = {"x": s.read_solution(pol), "ART": s.absorption(pol=pol)}
        if case["maps"]:
            got["per_tet"] = s.absorption_per_tet(pol)
            got["field"] = s.sample_field(state["points"], pol)
        out.append(got)
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def _sizes(case):
    """(unknowns, tetrahedra, unknowns per domain) of a case's mesh."""
    m = _mesh(case)
    n = W.count_unknowns_paired(*m.grid)
    share = np.bincount(m.tet_domain, minlength=m.ndom) / m.nt
    return n, m.nt, [n * float(f) for f in share]


def _fill_work(n, nt, entry):
    # Z written once; per unordered pair of tetrahedra 16 kernel values brought into two sets of moments (44 operations
    # each at the least) and the 2 x 16 entries formed from those (1,200 each way)
    return entry * n * n, nt * nt / 2 * (16 * 44 + 2400)


def _factor_work(doms, entry):
    return 2 * entry * sum(d * d for d in doms), 8 / 3 * sum(d ** 3 for d in doms)


def _solve_work(n, doms, entry, vectors):
    # each Krylov step reads Z and the factors once, for all its vectors
    each = n * n + sum(d * d for d in doms)
    return ITERS * entry * each, ITERS * 8 * each * vectors


def work(case):
    kind = case["kind"]
    entry = 8 if case.get("precision") == "mixed" else 16
    if kind == "pgf":
        return {"bytes": 40 * case["points"], "flops": 100 * case["points"]}
    parts = []
    if kind == "batch":
        cells = W.batch_cells(case["cells"], seed=case["cell_seed"], n_lo=case["n_lo"], n_hi=case["n_hi"])
        for c in cells:
            n, nt, doms = _sizes({"shape": "osc", **c})
            parts += [_fill_work(n, nt, entry), _factor_work(doms, entry), _solve_work(n, doms, entry, 1)]
    elif kind == "grid":
        m = _mesh(case)
        nx, ny, nz = (len(g) - 1 for g in m.grid)
        nf = nx * ny * 2 * (nz + 1)
        near = 188 * W.count_unknowns_paired(*m.grid)   # touching pairs: entries of the sparse part
        # a product reads the 60 x 60 kernel tables and the sparse part once; a fill writes them
        bytes_ = 16 * 3600 * nf + 20 * near
        parts = [(bytes_, 8 * (3600 + 3 * 24 * 24) * nf)]
        if not case["product_only"]:
            parts.append((bytes_, 3600 * nf * 100 + near * 1000))
    else:
        n, nt, doms = _sizes(case)
        if kind in ("request", "fill"):
            parts.append(_fill_work(n, nt, entry))
        if kind in ("request", "factor"):
            parts.append(_factor_work(doms, entry))
        if kind == "fill":
            parts.append((entry * n * n, 8 * n * n))
        elif kind == "factor":
            parts.append((entry * sum(d * d for d in doms), 8 * sum(d * d for d in doms)))
        else:
            parts.append(_solve_work(n, doms, entry, 2 if kind == "pair" or case["pair"] else 1))
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ------------------------------------------------------------------ values in 64 bits
def exact(case, seed):
    """The Green's function samples by an Ewald sum of its own.  The other kinds return values of the discrete
    problem (quadrature rules, singular extraction): they have no value outside this library but that of a second
    assembly of it, which the parity tests hold."""
    if case["kind"] != "pgf":
        return None
    rng = np.random.default_rng([seed, 77])
    lam, theta, phi = _wave(case, rng)
    _eps(case, _mesh(case), lam, rng)
    d = _separations(case, rng)
    a, k = case["a"], 2 * math.pi / lam
    kx, ky = k * math.sin(theta) * math.cos(phi), k * math.sin(theta) * math.sin(phi)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    x, y, z = (torch.from_numpy(np.ascontiguousarray(d[:, i])).to(dev) for i in range(3))
    z = z.abs()
    split = math.sqrt(math.pi) / a
    M = 6
    # images: G = 1 / (2 pi^1.5) int_0^inf exp(-R^2 s^2 + k^2 / 4 s^2) ds, here the part s > split
    m0, n0 = torch.round(x / a), torch.round(y / a)
    g = torch.zeros(len(x), dtype=torch.complex128, device=dev)
    for m in range(-M, M + 1):
        for n in range(-M, M + 1):
            mm, nn = m - m0, n - n0
            r = torch.sqrt((x + mm * a) ** 2 + (y + nn * a) ** 2 + z ** 2)
            g += torch.exp(1j * (kx * mm + ky * nn) * a) * (_tails(r, split, k * k, 0) / (2 * math.pi ** 1.5))
    # orders: int_0^split 1 / (2 sqrt(pi) s^2) exp(-z^2 s^2 - gamma^2 / 4 s^2) ds
    for p in range(-M, M + 1):
        for q in range(-M, M + 1):
            px, py = kx + 2 * math.pi * p / a, ky + 2 * math.pi * q / a
            g2 = px * px + py * py - k * k
            if g2 > 0:
                ga = math.sqrt(g2)
                u = ga / (2 * split)
                K = (torch.exp(ga * z) * torch.special.erfc(u + z * split)
                     + torch.exp(-ga * z) * torch.special.erfc(u - z * split)) / (4 * ga)
            else:   # propagating: the whole of it less the part s > split
                ga = 1j * math.sqrt(-g2)
                K = torch.exp(-ga * z) / (2 * ga) - _tails(z, split, -g2, 1) / (2 * math.sqrt(math.pi))
            g += torch.exp(-1j * (px * x + py * y)) * K / (a * a)
    return g.cpu().numpy()


def _tails(r, split, c, first):
    """int_split^inf s^(-2 first) exp(-r^2 s^2 + c / 4 s^2) ds by the powers of c: J_n = int s^(-2n) exp(-r^2 s^2) ds."""
    e = torch.exp(-(r * split) ** 2)
    j = torch.special.erfc(r * split) * (math.sqrt(math.pi) / 2) / torch.clamp(r, min=1e-300)
    total, coef = torch.zeros_like(r), 1.0
    for n in range(45):
        if n >= first:
            total = total + coef * j
            coef *= c / 4 / (n - first + 1)
        j = (e * split ** (-2 * n - 1) - 2 * r * r * j) / (2 * n + 1)
    return total
