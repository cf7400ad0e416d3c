"""GPU adjoint gradient of a far-field intensity with respect to the per-leaf
permittivity (hdp_far_intensity_gradient, and the torch.autograd wrapper),
against the oracle's adjoint (plain conforming solves) on a small design
problem, and against central finite differences of the GPU's own J at the
full 64x64 design-block size."""
import numpy as np
import pytest

import workloads as W
from oracle import adjoint as adj

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def hdp():
    import paper_1808_04713_amd as m
    return m


def design_case():
    w = W.small_uniform(6, 4, 6.0, domain=(-1.0, 1.0, -1.0, 1.0), l=2)
    c = W.leaf_centres(w)
    inside = (np.abs(c[:, 0]) < 0.4) & (np.abs(c[:, 1]) < 0.4)
    eps = np.where(inside, np.random.default_rng(3).uniform(1.0, 4.0, len(c)), 1.0)
    return dict(w, eps_r=eps), inside


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_gradient_matches_oracle_adjoint(precision):
    w, inside = design_case()
    J0, g0, E0 = adj.eps_gradient(w, 0.0, 0.0, inside)
    s = hdp().Solver(w, precision=precision, tol=1e-13, max_iter=400)
    J, g, st = s.far_intensity_gradient(0.0, 0.0, inside)
    s.close()
    assert st["converged"]
    tol = 1e-9 if precision == "fp64" else 1e-7
    assert abs(J - J0) < tol * J0
    assert np.linalg.norm(g - g0) < tol * np.linalg.norm(g0)


def test_gradient_with_two_boundary_sides_on_one_element():
    """A boundary around an L: the outside element in its notch carries two sides,
    which one workgroup adds."""
    w, _ = design_case()
    c = W.leaf_centres(w)
    inside = (np.abs(c[:, 0]) < 0.7) & (np.abs(c[:, 1]) < 0.7) & ~((c[:, 0] > 0.4) & (c[:, 1] > 0.4))
    J0, g0, E0 = adj.eps_gradient(w, 0.4, 2.1, inside)
    s = hdp().Solver(w, tol=1e-13, max_iter=400)
    J, g, st = s.far_intensity_gradient(0.4, 2.1, inside)
    s.close()
    assert abs(J - J0) < 1e-9 * J0
    assert np.linalg.norm(g - g0) < 1e-9 * np.linalg.norm(g0)


def test_autograd_function_returns_the_adjoint_gradient():
    w, inside = design_case()
    _, g0, _ = adj.eps_gradient(w, 0.0, 0.0, inside)
    eps = torch.tensor(w["eps_r"], dtype=torch.float64, requires_grad=True)
    J = hdp().far_intensity(eps, w, 0.0, 0.0, inside, tol=1e-13, max_iter=400)
    (3.0 * J).backward()
    assert np.linalg.norm(eps.grad.numpy() - 3.0 * g0) < 1e-9 * 3.0 * np.linalg.norm(g0)


def _design_block():
    w = W.design_block_64x64()
    c = W.leaf_centres(w)
    h_el = 2.0 / 64
    inside = (np.abs(c[:, 0]) < 8 * h_el) & (np.abs(c[:, 1]) < 8 * h_el)
    return w, inside


def test_full_size_design_block_against_oracle_adjoint():
    """64x64 elements, p = 12, k = 150, eps_r ~ U[1,4] on the central 16x16 block:
    J and all 256 design-parameter derivatives against the oracle's adjoint
    (element-wise dual-primal solves, stored by tests/golden/make_design_block_64x64.py).
    Both sides stop GMRES at a preconditioned relative residual of 1e-13, which
    bounds each state's relative error by kappa(P^-1 F) 1e-13 only.  J depends on
    the forward state alone and is held to 1e-9; each derivative is a bilinear
    form in the forward and the adjoint state (the adjoint solve starts from the
    forward field), so both states' errors enter it, and the gradient is held
    to 3e-8 in the 2-norm (the difference at full size is about 1e-8)."""
    import os
    path = os.path.join(os.path.dirname(__file__), "golden", "design_block_64x64_gradient.txt")
    ref = {}
    J0 = None
    for line in open(path):
        t = line.split()
        if t and t[0] == "J":
            J0 = float(t[1])
        elif t and t[0] == "grad":
            ref[int(t[1])] = float(t[2])
    w, inside = _design_block()
    s = hdp().Solver(w, tol=1e-13, max_iter=400)
    J, g, st = s.far_intensity_gradient(0.0, 0.0, inside)
    s.close()
    assert st["converged"]
    idx = sorted(ref)
    assert idx == list(np.nonzero(inside)[0])
    g0 = np.array([ref[e] for e in idx])
    assert abs(J - J0) < 1e-9 * J0
    assert np.linalg.norm(g[idx] - g0) < 3e-8 * np.linalg.norm(g0)


def test_full_size_design_block_against_central_differences():
    """Central differences of the GPU's J with step h = 1e-6 on 8 random design
    parameters.  A difference quotient carries the rounding noise of J between
    set-ups (each perturbed problem is set up and factored anew) divided by h;
    that noise delta is measured here by two set-ups of the unperturbed problem,
    and the comparison allows 1e-3 relative plus 4 delta / h."""
    w, inside = _design_block()
    opts = dict(tol=1e-13, max_iter=400)
    s = hdp().Solver(w, **opts)
    J, g, st = s.far_intensity_gradient(0.0, 0.0, inside)
    s.close()
    s = hdp().Solver(w, **opts)
    J_again = s.far_intensity_gradient(0.0, 0.0, inside)[0]
    s.close()
    delta = max(abs(J_again - J), 1e-15 * J)
    assert st["converged"] and J > 0
    idx = np.nonzero(inside)[0]
    assert len(idx) == 256
    rng = np.random.default_rng(11)
    h = 1e-6
    for e in rng.choice(idx, 8, replace=False):
        Js = []
        for sgn in (1, -1):
            eps = w["eps_r"].copy()
            eps[e] += sgn * h
            s2 = hdp().Solver(dict(w, eps_r=eps), **opts)
            Js.append(s2.far_intensity_gradient(0.0, 0.0, inside)[0])
            s2.close()
        fd = (Js[0] - Js[1]) / (2 * h)
        assert abs(fd - g[e]) < 1e-3 * abs(g[e]) + 4 * delta / h, (e, fd, g[e], delta)
