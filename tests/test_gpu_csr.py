"""GPU global assembly (coffee_csr_pattern, coffee_assemble_csr) against the
oracle's plain global assembler (element tensors scattered into a coordinate
list, duplicates summed by scipy): the CSR pattern is compared exactly, the
values row by row."""
import numpy as np
import pytest

from paper_1407_0904_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cf():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a device"
    from paper_1407_0904_amd import coffee
    return coffee


def _space(mesh, p):
    if p == 1:
        return mesh.cells, mesh.nvert
    return I.p2_dofmap(mesh.cells, mesh.n, mesh.d)


def _row_rel_err(vals, indptr, ref):
    """max over rows of max |got - ref| / max |ref row| (ref a scipy CSR)."""
    err = 0.0
    d = np.abs(vals - ref.data)
    for r in range(len(indptr) - 1):
        a, b = indptr[r], indptr[r + 1]
        if b > a:
            err = max(err, d[a:b].max() / max(np.abs(ref.data[a:b]).max(), 1e-300))
    return err


CASES = [
    # form, d, p, n (mesh), fields
    ("mass", 2, 1, 9, "p1"), ("helmholtz", 3, 2, 3, "p2"), ("elasticity", 3, 2, 3, "lame"),
    ("burgers", 3, 1, 3, "w1"), ("svk_jacobian", 3, 2, 2, "u2"), ("helmholtz", 2, 3, 5, "cellmajor"),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("form,d,p,n,kind", CASES)
def test_csr_vs_oracle(cf, oracle, form, d, p, n, kind, prec):
    import torch
    from gpu_util import TOL, to_dev
    rng = np.random.default_rng(17 + 3 * p + d)
    mesh = I.make_mesh(d, n, 0.12, rng)
    cst = []
    if kind == "p1":
        fields = [I.Field(rng.uniform(0.5, 1.5, (mesh.nvert, 1)), mesh.cells, 1, 1)]
    elif kind == "p2":
        c2d, nd = I.p2_dofmap(mesh.cells, mesh.n, d)
        fields = [I.Field(rng.uniform(0.5, 1.5, (nd, 1)), c2d, 2, 1)]
    elif kind == "lame":
        fields = [I.Field(rng.uniform(1, 10, (mesh.nvert, 1)), mesh.cells, 1, 1) for _ in range(2)]
    elif kind == "w1":
        fields = [I.Field(rng.uniform(-1, 1, (mesh.nvert, d)), mesh.cells, 1, d)]
        cst = [0.7, 1.3]
    elif kind == "u2":
        c2d, nd = I.p2_dofmap(mesh.cells, mesh.n, d)
        fields = [I.Field(rng.normal(0, 0.05, (nd, d)), c2d, 2, d)]
        cst = [1.1, 0.9]
    else:  # a cell-major P2 coefficient field (no map); the space is discontinuous P3 per cell
        fields = [I.Field(rng.uniform(0.5, 1.5, (mesh.ncells, 6, 1)), None, 2, 1)]
    if kind == "cellmajor":
        nl = I.n_scalar_dofs(d, p)
        c2d, nd = np.arange(mesh.ncells * nl, dtype=np.int32).reshape(mesh.ncells, nl), mesh.ncells * nl
    else:
        c2d, nd = _space(mesh, p)
    ref = oracle.assemble_global(form, mesh, p, c2d, nd, fields=fields, constants=cst)
    coords, c2v, dfs = to_dev(mesh, fields)
    map_d = torch.as_tensor(np.ascontiguousarray(c2d, dtype=np.int32), device=coords.device)
    N = oracle.tensor_dim(form, d, p)
    ncomp = N // c2d.shape[1]
    row_ptr, col_idx = cf.coffee_csr_pattern(map_d, nd, ncomp)
    np.testing.assert_array_equal(row_ptr.cpu().numpy(), ref.indptr)
    np.testing.assert_array_equal(col_idx.cpu().numpy(), ref.indices)
    vals = cf.coffee_assemble_csr(form, d, p, coords, c2v, row_ptr, col_idx, nd, cell_to_dof=map_d, coeffs=dfs,
                                  constants=cst, precision=prec)
    torch.cuda.synchronize()
    err = _row_rel_err(vals.cpu().numpy().astype(np.float64), ref.indptr, ref)
    print(f"csr {form} d{d} p{p} {prec}: nnz {ref.nnz}, row rel err {err:.3e}")
    # sums of element entries: the element tolerance, with a few entries per sum
    assert err < 4 * TOL[prec]


def test_csr_several_chunks(cf, oracle):
    """131,712 P1 tetrahedra (more than one 131,072-cell chunk) assembled into
    the global Helmholtz matrix; against the oracle, and the global mass
    (f = 1) sums to the cube's volume."""
    import torch
    from gpu_util import to_dev
    rng = np.random.default_rng(4)
    mesh = I.make_mesh(3, 28, 0.1, rng)
    assert mesh.ncells > 131072
    f = [I.Field(rng.uniform(0.5, 1.5, (mesh.nvert, 1)), mesh.cells, 1, 1)]
    ref = oracle.assemble_global("helmholtz", mesh, 1, mesh.cells, mesh.nvert, fields=f)
    coords, c2v, dfs = to_dev(mesh, f)
    row_ptr, col_idx = cf.coffee_csr_pattern(c2v, mesh.nvert)
    np.testing.assert_array_equal(col_idx.cpu().numpy(), ref.indices)
    vals = cf.coffee_assemble_csr("helmholtz", 3, 1, coords, c2v, row_ptr, col_idx, mesh.nvert, coeffs=dfs)
    torch.cuda.synchronize()
    assert _row_rel_err(vals.cpu().numpy(), ref.indptr, ref) < 1e-12
    m = cf.coffee_assemble_csr("mass", 3, 1, coords, c2v, row_ptr, col_idx, mesh.nvert)
    assert abs(float(m.sum()) - 1.0) < 1e-10


def test_csr_pattern_edge_cases(cf):
    """An empty mesh gives an empty pattern with zero row pointers; a too
    small column buffer is reported with the count."""
    import ctypes as C
    import torch
    dev = torch.device("cuda:0")
    empty = torch.empty((0, 3), dtype=torch.int32, device=dev)
    row_ptr, col_idx = cf.coffee_csr_pattern(empty, 5)
    assert col_idx.numel() == 0 and torch.all(row_ptr == 0)
    mesh = I.make_mesh(2, 3, 0.1, np.random.default_rng(0))
    c2v = torch.as_tensor(mesh.cells, device=dev)
    nnz_expected = (3 + 1) ** 2 + 2 * (3 * 9 + 6)
    rp, ci = cf.coffee_csr_pattern(c2v, mesh.nvert)
    assert ci.numel() == nnz_expected
    ws = torch.empty(cf._lib.coffee_csr_pattern_workspace_size(mesh.ncells, 3, mesh.nvert), dtype=torch.uint8,
                     device=dev)
    nnz = C.c_int64()
    small = torch.empty(10, dtype=torch.int32, device=dev)
    st = cf._lib.coffee_csr_pattern(c2v.data_ptr(), mesh.ncells, 3, mesh.nvert, 1, rp.data_ptr(), small.data_ptr(),
                                    10, C.byref(nnz), ws.data_ptr(), ws.numel(), None)
    assert st == 3 and nnz.value == nnz_expected


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("form,d,p,n", [("helmholtz", 3, 2, 5), ("elasticity", 3, 2, 3), ("mass", 3, 1, 9),
                                        ("mass", 2, 3, 11), ("elasticity", 2, 2, 7), ("helmholtz", 3, 3, 2)])
def test_csr_runs_of_scattered_cells(cf, oracle, form, d, p, n, prec):
    """Cells in random order (runs with more dofs than the LDS matrix has rows are split), counts that leave a
    partial run, and a pattern that holds more entries than the assembled cells fill."""
    import torch
    from gpu_util import TOL, to_dev
    rng = np.random.default_rng(5 + n)
    mesh = I.make_mesh(d, n, 0.12, rng)
    if p == 3:  # every cell its own dofs, then shared at random: any map is a valid space for the scatter
        nd = mesh.ncells * 3
        nl = 10 if d == 2 else 20
        c2d = np.stack([rng.permutation(nd)[:nl] for _ in range(mesh.ncells)]).astype(np.int32)
    else:
        c2d, nd = _space(mesh, p)
    order = rng.permutation(mesh.ncells)
    cells, c2d = np.ascontiguousarray(mesh.cells[order]), np.ascontiguousarray(c2d[order])
    cst = [1.5, 0.5] if form == "elasticity" else []
    nc = d if form == "elasticity" else 1
    coords, c2v, _ = to_dev(I.Mesh(d, n, mesh.coords, cells), [])
    dofs = torch.as_tensor(c2d, device=coords.device)
    row_ptr, col_idx = cf.coffee_csr_pattern(dofs, nd, nc)
    rp, ci = row_ptr.cpu().numpy(), col_idx.cpu().numpy()
    for count in (1, 7, mesh.ncells - 1, mesh.ncells):
        sub = I.Mesh(d, n, mesh.coords, np.ascontiguousarray(cells[:count]))
        A = oracle.assemble(form, sub, p, constants=cst)
        got = cf.coffee_assemble_csr(form, d, p, coords, c2v[:count].contiguous(), row_ptr, col_idx, nd,
                                     cell_to_dof=dofs[:count].contiguous(), constants=cst, precision=prec).cpu().numpy()
        g = np.concatenate([c2d[:count].astype(np.int64) * nc + c for c in range(nc)], axis=1)
        keys = np.repeat(np.arange(nd * nc), np.diff(rp)) * (nd * nc) + ci
        ref = np.zeros(len(ci))
        np.add.at(ref, np.searchsorted(keys, (g[:, :, None] * (nd * nc) + g[:, None, :]).ravel()), A.ravel())
        # entries are sums of at most a few dozen tensor values of that size
        assert np.abs(got - ref).max() <= 10 * TOL[prec] * np.abs(A).max(), count


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("form,cells", [("mass", 1021), ("mass", 1026), ("helmholtz", 5003), ("elasticity", 511),
                                        ("elasticity", 2001)])
def test_csr_long_rows(cf, oracle, form, cells, prec):
    """A fan of triangles around one vertex: its matrix row has a column for every vertex (cells + 2, times two in
    elasticity), below and above the length from which the run's columns are searched in a row, and the rest are
    short."""
    import torch
    from gpu_util import TOL, to_dev
    t = np.linspace(0, 1.5 * np.pi, cells + 1)
    x = np.concatenate([np.zeros((1, 2)), np.stack([np.cos(t), np.sin(t)], 1)])
    i = np.arange(cells)
    mesh = I.Mesh(2, 1, x, np.stack([0 * i, i + 1, i + 2], 1).astype(np.int32))
    cst = [1.5, 0.5] if form == "elasticity" else []
    nc = 2 if form == "elasticity" else 1
    ref = oracle.assemble_global(form, mesh, 1, mesh.cells, mesh.nvert, constants=cst)
    coords, c2v, _ = to_dev(mesh, [])
    row_ptr, col_idx = cf.coffee_csr_pattern(c2v, mesh.nvert, nc)
    assert int(row_ptr[1]) == nc * (cells + 2)
    np.testing.assert_array_equal(col_idx.cpu().numpy(), ref.indices)
    vals = cf.coffee_assemble_csr(form, 2, 1, coords, c2v, row_ptr, col_idx, mesh.nvert, constants=cst, precision=prec)
    torch.cuda.synchronize()
    got = vals.cpu().numpy()
    # the hub's diagonal sums `cells` entries of one sign, in runs: rounding grows with the number of sums
    scale = np.abs(ref.data).max()
    assert np.abs(got - ref.data).max() <= 4 * TOL[prec] * scale
    short = np.repeat(np.diff(ref.indptr), np.diff(ref.indptr)) <= 1024
    assert np.abs(got - ref.data)[short].max() <= 4 * TOL[prec] * np.abs(ref.data[short]).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("form,cell,p", [
    ("mass", "triangle", 1), ("mass", "triangle", 2), ("mass", "triangle", 3), ("mass", "triangle", 4),
    ("elasticity", "triangle", 1), ("elasticity", "triangle", 2), ("elasticity", "triangle", 3),
    ("mass", "tetrahedron", 1), ("mass", "tetrahedron", 2), ("mass", "tetrahedron", 3), ("mass", "tetrahedron", 4),
    ("elasticity", "tetrahedron", 1), ("elasticity", "tetrahedron", 2), ("elasticity", "tetrahedron", 3),
    ("mass", "prism", 1), ("mass", "prism", 2)])
def test_csr_long_and_short_runs(cf, oracle, form, cell, p, shuffled, prec):
    """Every space, at the largest count that takes the runs that always fit (90 dof rows, two workgroups per CU) and
    a few cells more, which take the long ones: cells in mesh order, and in random order (long runs are split)."""
    import torch
    from gpu_util import TOL, to_dev
    d = 2 if cell == "triangle" else 3
    nc = d if form == "elasticity" else 1
    nl = {"triangle": (p + 1) * (p + 2) // 2, "tetrahedron": (p + 1) * (p + 2) * (p + 3) // 6,
          "prism": (p + 1) * (p + 2) // 2 * (p + 1)}[cell]
    most = 90 // nc // nl * 2 * torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(800 + 10 * d + p)
    n = int(np.ceil(((most + 5) / {"triangle": 2, "tetrahedron": 6, "prism": 2}[cell]) ** (1 / d)))
    mesh = I.make_prism_mesh(n, 0.1, rng) if cell == "prism" else I.make_mesh(d, n, 0.1, rng)
    if p == 1:
        c2d, nd = mesh.cells, mesh.nvert
    elif p == 2 and cell != "prism":
        c2d, nd = I.p2_dofmap(mesh.cells, mesh.n, d)
    else:  # distinct dofs per cell, shared by neighbours in number: any map is a valid space for the scatter
        nd = mesh.ncells * nl // 5 + 2 * nl
        c2d = (np.arange(mesh.ncells)[:, None] * (nl // 5 + 1) + np.arange(nl)[None, :]) % nd
    order = rng.permutation(mesh.ncells) if shuffled else np.arange(mesh.ncells)
    cells = np.ascontiguousarray(mesh.cells[order])
    c2d = np.ascontiguousarray(np.asarray(c2d, dtype=np.int32)[order])
    cst = [1.5, 0.5] if form == "elasticity" else []
    coords, c2v, _ = to_dev(I.Mesh(d, n, mesh.coords, cells), [])
    code = {"triangle": 2, "tetrahedron": 3, "prism": 6}[cell]
    dofs = torch.as_tensor(c2d, device=coords.device)
    row_ptr, col_idx = cf.coffee_csr_pattern(dofs, nd, nc)
    rp, ci = row_ptr.cpu().numpy(), col_idx.cpu().numpy()
    A = oracle.assemble(form, I.Mesh(d, n, mesh.coords, np.ascontiguousarray(cells[:most + 5])), p, constants=cst)
    keys = np.repeat(np.arange(nd * nc), np.diff(rp)) * (nd * nc) + ci
    g = np.concatenate([c2d[:most + 5].astype(np.int64) * nc + c for c in range(nc)], axis=1)
    for count in (most, most + 5):
        got = cf.coffee_assemble_csr(form, code, p, coords, c2v[:count].contiguous(), row_ptr, col_idx, nd,
                                     cell_to_dof=dofs[:count].contiguous(), constants=cst, precision=prec).cpu().numpy()
        ref = np.zeros(len(ci))
        at = np.searchsorted(keys, (g[:count, :, None] * (nd * nc) + g[:count, None, :]).ravel())
        np.add.at(ref, at, A[:count].ravel())
        # entries are sums of at most a few dozen tensor values of that size
        assert np.abs(got - ref).max() <= 10 * TOL[prec] * np.abs(A).max(), count


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("form,cell,p,half", [
    ("mass", "triangle", 1, 43), ("mass", "triangle", 3, 7), ("elasticity", "triangle", 1, 21),
    ("mass", "tetrahedron", 1, 57), ("mass", "tetrahedron", 2, 10), ("elasticity", "tetrahedron", 1, 15),
    ("mass", "prism", 1, 14), ("mass", "prism", 2, 4)])
def test_csr_runs_of_half_length(cf, oracle, form, cell, p, half, prec, shuffled):
    """Meshes between those of the shortest and of the longest runs: the largest count whose runs of half the cells are
    all resident (two workgroups per CU) and one cell more; the matrix against the sum of the oracle's tensors."""
    import torch
    from gpu_util import TOL, to_dev
    d = 2 if cell == "triangle" else 3
    nc = d if form == "elasticity" else 1
    nl = {"triangle": (p + 1) * (p + 2) // 2, "tetrahedron": (p + 1) * (p + 2) * (p + 3) // 6,
          "prism": (p + 1) * (p + 2) // 2 * (p + 1)}[cell]
    most = half * 2 * torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(900 + 10 * d + p)
    n = int(np.ceil(((most + 1) / {"triangle": 2, "tetrahedron": 6, "prism": 2}[cell]) ** (1 / d)))
    mesh = I.make_prism_mesh(n, 0.1, rng) if cell == "prism" else I.make_mesh(d, n, 0.1, rng)
    if p == 1:
        c2d, nd = mesh.cells, mesh.nvert
    else:  # distinct dofs per cell, shared by neighbours in number: any map is a valid space for the scatter
        nd = mesh.ncells * nl // 5 + 2 * nl
        c2d = (np.arange(mesh.ncells)[:, None] * (nl // 5 + 1) + np.arange(nl)[None, :]) % nd
    order = rng.permutation(mesh.ncells) if shuffled else np.arange(mesh.ncells)
    cells = np.ascontiguousarray(mesh.cells[order][:most + 1])
    c2d = np.ascontiguousarray(np.asarray(c2d, dtype=np.int32)[order][:most + 1])
    cst = [1.5, 0.5] if form == "elasticity" else []
    coords, c2v, _ = to_dev(I.Mesh(d, n, mesh.coords, cells), [])
    code = {"triangle": 2, "tetrahedron": 3, "prism": 6}[cell]
    dofs = torch.as_tensor(c2d, device=coords.device)
    row_ptr, col_idx = cf.coffee_csr_pattern(dofs, nd, nc)
    rp, ci = row_ptr.cpu().numpy(), col_idx.cpu().numpy()
    A = oracle.assemble(form, I.Mesh(d, n, mesh.coords, cells), p, constants=cst)
    keys = np.repeat(np.arange(nd * nc), np.diff(rp)) * (nd * nc) + ci
    g = np.concatenate([c2d.astype(np.int64) * nc + c for c in range(nc)], axis=1)
    at = np.searchsorted(keys, (g[:, :, None] * (nd * nc) + g[:, None, :]).ravel()).reshape(len(g), -1)
    for count in (most, most + 1):
        got = cf.coffee_assemble_csr(form, code, p, coords, c2v[:count].contiguous(), row_ptr, col_idx, nd,
                                     cell_to_dof=dofs[:count].contiguous(), constants=cst, precision=prec).cpu().numpy()
        ref = np.bincount(at[:count].ravel(), weights=A[:count].reshape(count, -1).ravel(), minlength=len(ci))
        # entries share a cell's largest entry as their scale; sums of up to a few dozen of them per nonzero
        assert np.abs(got - ref).max() <= 4 * TOL[prec] * np.abs(ref).max()
