"""GPU checks of the separable element solve (Sec. 2.2.1, remark on the fast
solver) through the C ABI: X = Ex [(Ex^T Y Ey) ./ D] Ey^T on every element,
on the matrix cores for classes of at most 32 modes per direction (real
eigenbasis on interior elements, complex on impedance-boundary elements) and on
the vector ALUs above, against dense solves of each element matrix, at column
counts that exercise every column-block width; and the element solves of the
interface right-hand side and the recovery (coarse pass, coarse solve,
corrected full solve) against the oracle's block elimination."""
import numpy as np
import pytest

import workloads as W
from oracle import dp, dp_elementwise as dpe, element as el, problem as pb

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def hdp():
    import paper_1808_04713_amd as m
    return m


def rel(a, b):
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b))


def _mixed_degrees():
    """4x4 mesh with degrees 2..12 (several classes, real and complex bases)."""
    w = W.small_uniform(4, 6, 9.0, l=2)
    w["degree"] = np.random.default_rng(11).integers(2, 13, 16)
    return w


def _dense_ref(w, y):
    disc = pb.Discretisation(w)
    out = np.zeros_like(y)
    off = 0
    for e in range(disc.mesh.E):
        n = int(disc.degrees[e]) + 1
        B = el.to_vertex_basis(n)
        A = B @ disc.A[e] @ B
        out[off:off + n * n] = np.linalg.solve(A, y[off:off + n * n])
        off += n * n
    return out


@pytest.mark.parametrize("R", [1, 3, 8, 16, 64])
def test_local_solve_all_widths(R):
    w = _mixed_degrees()
    s = hdp().Solver(w, max_rhs=min(R, 64))
    rng = np.random.default_rng(R)
    y = rng.standard_normal((s.dof, R)) + 1j * rng.standard_normal((s.dof, R))
    print(f"local solve R={R}", flush=True)
    x = s.local_solve(torch.from_numpy(y).cuda()).cpu().numpy()
    assert rel(x, _dense_ref(w, y)) < 1e-11
    s.close()


@pytest.mark.parametrize("cols", [1, 2, 4, 8, 16])
def test_local_solve_every_tile_width(cols):
    w = _mixed_degrees()
    s = hdp().Solver(w, max_rhs=16, tile_fdm=cols)
    rng = np.random.default_rng(cols)
    y = rng.standard_normal((s.dof, 16)) + 1j * rng.standard_normal((s.dof, 16))
    x = s.local_solve(torch.from_numpy(y).cuda()).cpu().numpy()
    assert rel(x, _dense_ref(w, y)) < 1e-11
    s.close()


def test_autotuner_table_and_tuned_solve():
    """HDP_FLAG_AUTOTUNE times every tile width that fits and keeps the fastest;
    the tuned solver gives the same field as the untuned one."""
    w = _mixed_degrees()
    kind, vals = hdp().rhs_values(w)
    vals16 = np.linspace(0.0, 2 * np.pi, 16, endpoint=False)
    st = hdp().Solver(w, max_rhs=16, tol=1e-12, autotune=True)
    su = hdp().Solver(w, max_rhs=16, tol=1e-12)
    tab = st.autotune_table()
    fams = {t["kernel"] for t in tab}
    assert fams == {"fdm_element_solve", "slot_operator"}
    for fam in fams:
        rows = [t for t in tab if t["kernel"] == fam]
        assert sum(t["chosen"] for t in rows) == 1
        best = min(rows, key=lambda t: t["ms"])
        assert best["chosen"] and best["ms"] > 0
    assert {t["cols"] for t in tab if t["kernel"] == "fdm_element_solve"} == {1, 2, 4, 8, 16}
    a, _ = st.solve("plane_wave_total", vals16)
    b, _ = su.solve("plane_wave_total", vals16)
    assert rel(a.cpu().numpy(), b.cpu().numpy()) < 1e-10
    assert su.autotune_table() == []
    st.close()
    su.close()


def test_local_solve_above_32_modes():
    """p = 34 (35 modes): the vector-ALU separable solve."""
    w = W.small_uniform(2, 34, 5.0, l=2)
    s = hdp().Solver(w)
    rng = np.random.default_rng(3)
    y = rng.standard_normal((s.dof, 2)) + 1j * rng.standard_normal((s.dof, 2))
    x = s.local_solve(torch.from_numpy(y).cuda()).cpu().numpy()
    assert rel(x, _dense_ref(w, y)) < 1e-10
    s.close()


@pytest.mark.parametrize("make", [_mixed_degrees, lambda: W.small_uniform(2, 34, 5.0, l=2)])
def test_interface_rhs_and_field_of_mixed_degrees(make):
    """The interface right-hand side (first element solve) and the field (the
    recovery) on a mesh of uneven degree, FP64, against the literal oracle."""
    w = make()
    disc = pb.Discretisation(w)
    l = pb.coarse_order(w, disc.mesh)
    D = dp.LiteralDP(disc, l)
    s = hdp().Solver(w, tol=1e-12, max_iter=300)
    kind, vals = hdp().rhs_values(w)
    g = s.interface_rhs(kind, vals).cpu().numpy()[:, 0]
    assert rel(g, D.g) < 1e-11
    field, st = s.solve(kind, vals)
    phis = D.solve(tol=1e-12, max_iter=300)
    ref = np.concatenate(pb.gll_field(disc.mesh, disc.degrees, phis))
    assert rel(field.cpu().numpy()[0], ref) < 1e-10
    s.close()


@pytest.mark.parametrize("p", [1, 2, 3, 4, 7, 8, 11, 12, 15, 16, 17, 18, 19, 20, 21, 22, 23, 24, 28, 32])
def test_local_solve_at_the_edges_of_every_kernel(p):
    """Every number of modes at which the steps, row tiles or extra rows of the
    separable kernels change, on a mesh with interior, edge and corner elements
    (real, mixed and complex eigenbases), one column (several elements per
    workgroup) and five; the tolerance is cond(E_x) cond(E_y) eps."""
    w = W.small_uniform(4, p, 2.0 * p ** 0.5, l=1)
    s = hdp().Solver(w)
    for R in (1, 5):
        rng = np.random.default_rng(p)
        y = rng.standard_normal((s.dof, R)) + 1j * rng.standard_normal((s.dof, R))
        x = s.local_solve(torch.from_numpy(y).cuda()).cpu().numpy()
        assert rel(x, _dense_ref(w, y)) < 1e-10, R
    s.close()


def test_a_width_that_does_not_fit_a_compute_unit():
    """24 modes, 64 of them coarse: 16 columns of an element and the kernel's own array
    pass a compute unit's shared memory by that array.  Asked for, the size rule takes
    over; the autotuner leaves the width out.  cond(E_x) cond(E_y) eps as above."""
    w = W.small_uniform(2, 23, 9.0, l=16)
    rng = np.random.default_rng(23)
    s = hdp().Solver(w, max_rhs=16, tile_fdm=16)
    y = rng.standard_normal((s.dof, 16)) + 1j * rng.standard_normal((s.dof, 16))
    x = s.local_solve(torch.from_numpy(y).cuda()).cpu().numpy()
    assert rel(x, _dense_ref(w, y)) < 1e-10
    s.close()
    angles = np.linspace(0.0, 6.0, 16)
    st = hdp().Solver(w, max_rhs=16, autotune=True)
    assert {t["cols"] for t in st.autotune_table() if t["kernel"] == "fdm_element_solve"} == {1, 2, 4, 8}
    su = hdp().Solver(w, max_rhs=16)
    a, b = st.interface_rhs("plane_wave_total", angles), su.interface_rhs("plane_wave_total", angles)
    assert rel(a.cpu().numpy(), b.cpu().numpy()) < 1e-10
    st.close()
    su.close()


@pytest.mark.parametrize("p", [20, 22, 23, 24, 26, 27, 28, 30, 31])
def test_one_column_and_single_last_columns_of_two_row_tiles(p):
    """21 to 32 modes: four waves share a workgroup's only column by lines and rows, the
    only column of a last, narrower chunk with as many waves as the others' columns have
    tiles.  Columns of one call against the same columns one at a time (every sum in
    the same order: equal to the last bit) and against dense solves."""
    w = W.small_uniform(3, p, 2.0 * p ** 0.5, l=1)
    rng = np.random.default_rng(p)
    for cols in (0, 2, 4):
        s = hdp().Solver(w, tile_fdm=cols)
        y = rng.standard_normal((s.dof, 5)) + 1j * rng.standard_normal((s.dof, 5))
        yd = torch.from_numpy(y).cuda()
        x = s.local_solve(yd)
        ones = torch.cat([s.local_solve(yd[:, r:r + 1].contiguous()) for r in range(5)], dim=1)
        assert torch.equal(x, ones), cols
        assert rel(x.cpu().numpy(), _dense_ref(w, y)) < 1e-10, cols
        s.close()


def _every_kernel():
    """16 elements of 16 kernels or more: the smaller ones' few workgroups run in one
    launch, those of more than 32 modes in their own."""
    w = W.small_uniform(4, 6, 9.0, l=1)
    w["degree"] = np.array([1, 3, 5, 9, 12, 15, 16, 18, 20, 22, 26, 28, 31, 33, 35, 37])
    return w


@pytest.mark.parametrize("R", [1, 2, 5, 64, 720])
def test_local_solve_of_every_kernel_in_one_mesh(R):
    """Columns from one to so many that the small kernels run one after the other (2,048
    workgroups); the tolerance is cond(E_x) cond(E_y) eps."""
    w = _every_kernel()
    s = hdp().Solver(w)
    rng = np.random.default_rng(R)
    y = rng.standard_normal((s.dof, R)) + 1j * rng.standard_normal((s.dof, R))
    x = s.local_solve(torch.from_numpy(y).cuda()).cpu().numpy()
    ref = _dense_ref(w, y)
    off = np.concatenate([[0], np.cumsum((np.asarray(w["degree"]) + 1) ** 2)])
    for a, b in zip(off[:-1], off[1:]):
        assert rel(x[a:b], ref[a:b]) < 1e-10
    s.close()


@pytest.mark.parametrize("p", [27, 31, 33, 35, 36, 39, 40])
def test_local_solve_at_the_edges_of_the_largest_kernels(p):
    """The numbers of modes above 24 at which a kernel's last step, tile or row is full or
    begins, up to the largest degree, on corner, side and interior elements (complex,
    mixed and real eigenbases), one column and five; cond(E_x) cond(E_y) eps."""
    w = W.small_uniform(3, p, 2.0 * p ** 0.5, l=1)
    s = hdp().Solver(w)
    rng = np.random.default_rng(p)
    y = rng.standard_normal((s.dof, 5)) + 1j * rng.standard_normal((s.dof, 5))
    yd = torch.from_numpy(y).cuda()
    x = torch.cat([s.local_solve(yd), s.local_solve(yd[:, :1].contiguous())], dim=1).cpu().numpy()
    ref = _dense_ref(w, y)
    assert rel(x[:, :5], ref) < 1e-10
    assert rel(x[:, 5], ref[:, 0]) < 1e-10
    s.close()


def test_interface_rhs_and_field_above_36_modes():
    """Degrees 40, 36, 38 and 9: the coarse pass, the corrected solve and the GLL sampling
    of the kernels of three row tiles, beside a small one, against the literal oracle."""
    w = W.small_uniform(2, 9, 5.0, l=2)
    w["degree"] = np.array([40, 36, 38, 9])
    disc = pb.Discretisation(w)
    D = dp.LiteralDP(disc, pb.coarse_order(w, disc.mesh))
    s = hdp().Solver(w, tol=1e-12, max_iter=300)
    kind, vals = hdp().rhs_values(w)
    assert rel(s.interface_rhs(kind, vals).cpu().numpy()[:, 0], D.g) < 1e-11
    field, st = s.solve(kind, vals)
    ref = np.concatenate(pb.gll_field(disc.mesh, disc.degrees, D.solve(tol=1e-12, max_iter=300)))
    assert rel(field.cpu().numpy()[0], ref) < 1e-10
    s.close()
