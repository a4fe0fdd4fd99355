"""GPU St Venant-Kirchhoff energy, residual and Jacobian against the oracle,
and the energy's reverse pass against the oracle's complex-step gradient."""
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


def _disp(mesh, p, rng, sigma=0.05):
    d = mesh.d
    if p == 1:
        return I.Field(rng.normal(0, sigma, (mesh.nvert, d)), mesh.cells, 1, d)
    c2d, nd = I.p2_dofmap(mesh.cells, mesh.n, d)
    return I.Field(rng.normal(0, sigma, (nd, d)), c2d, 2, d)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("form", ["svk_energy", "svk_residual", "svk_jacobian"])
@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 1), (2, 2)])
def test_svk_forward(cf, oracle, form, d, p, prec):
    from gpu_util import TOL, assemble_gpu, cell_rel_err
    rng = np.random.default_rng(50 + 10 * d + p)
    mesh = I.make_mesh(d, 9 if d == 2 else 4, 0.1, rng)
    u = _disp(mesh, p, rng)
    cst = [1.3, 0.7]
    ref = oracle.assemble(form, mesh, p, fields=[u], constants=cst)
    got = assemble_gpu(form, mesh, p, [u], constants=cst, precision=prec).cpu().numpy()
    err = cell_rel_err(got.reshape(ref.shape[0], -1), ref.reshape(ref.shape[0], -1))
    print(f"{form} d{d} p{p} {prec}: {err:.3e}")
    assert err < TOL[prec]


@pytest.mark.parametrize("form", ["svk_energy", "svk_residual", "svk_jacobian"])
@pytest.mark.parametrize("d,p", [(3, 2), (3, 1), (2, 2)])
def test_svk_bf16x3_ragged_counts(cf, oracle, form, d, p):
    """BF16X3 SVK at cell counts around the 16-cell tile and the Jacobian's
    staging rounds, with the displacement through a dof map and cell-major."""
    from gpu_util import TOL, assemble_gpu, cell_rel_err
    rng = np.random.default_rng(90 + 10 * d + p)
    mesh = I.make_mesh(d, 9 if d == 2 else 4, 0.1, rng)
    u = _disp(mesh, p, rng)
    ucm = I.Field(np.ascontiguousarray(u.values[u.cell_to_dof]), None, u.degree, u.ncomp)
    cst = [1.1, 0.9]
    for count in (1, 7, 15, 16, 17, 40, 131):
        sub = I.Mesh(mesh.d, mesh.n, mesh.coords, np.ascontiguousarray(mesh.cells[:count]))
        ref = oracle.assemble(form, mesh, p, fields=[u], constants=cst, cells=np.arange(count))
        mapped = I.Field(u.values, np.ascontiguousarray(u.cell_to_dof[:count]), u.degree, u.ncomp)
        cellmajor = I.Field(np.ascontiguousarray(ucm.values[:count]), None, u.degree, u.ncomp)
        for f in (mapped, cellmajor):
            got = assemble_gpu(form, sub, p, [f], constants=cst, precision="bf16x3").cpu().numpy()
            err = cell_rel_err(got.reshape(count, -1), ref.reshape(count, -1))
            assert err < TOL["bf16x3"], (count, f.cell_to_dof is None, err)


@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 2)])
def test_svk_energy_adjoint(cf, oracle, d, p):
    import torch
    from gpu_util import to_dev
    rng = np.random.default_rng(60 + p)
    mesh = I.make_mesh(d, 6 if d == 2 else 3, 0.1, rng)
    u = _disp(mesh, p, rng)
    cst = [1.1, 0.9]
    S_ref, gc_ref, gu_ref = oracle.adjoint("svk_energy", mesh, p, fields=[u], constants=cst)
    coords, c2v, dfs = to_dev(mesh, [u])
    cv = torch.empty(mesh.ncells, dtype=torch.float64, device=coords.device)
    gc, gu = cf.coffee_assemble_adjoint("svk_energy", d, p, coords, c2v, coeffs=dfs, constants=cst, seed=1.0,
                                        cell_value=cv)
    torch.cuda.synchronize()
    S = float(cv.sum())
    gc = gc.cpu().numpy()
    gu = gu[0].cpu().numpy()
    rel = lambda a, b: float(np.max(np.abs(a - b)) / np.max(np.abs(b)))
    print(f"svk energy adjoint d{d} p{p}: S {abs(S - S_ref) / abs(S_ref):.2e} coords {rel(gc, gc_ref):.2e} "
          f"u {rel(gu, gu_ref[0]):.2e}")
    assert abs(S - S_ref) < 1e-11 * abs(S_ref)
    assert rel(gc, gc_ref) < 1e-10
    assert rel(gu, gu_ref[0]) < 1e-10


def test_svk_full_size_sampled(cf, oracle):
    """196,608-cell SVK P2 tetrahedra (u ~ N(0, 0.01)): sampled cells of all three outputs."""
    import torch
    from gpu_util import TOL, cell_rel_err, to_dev
    w = I.workload("svk_p2_tet")
    coords, c2v, dfs = to_dev(w.mesh, w.fields)
    rng = np.random.default_rng(5)
    E = w.mesh.ncells
    sample = np.unique(np.concatenate([[0, E - 1], rng.integers(0, E, 1000)]))
    idx = torch.as_tensor(sample, device=coords.device)
    for form in ("svk_energy", "svk_residual", "svk_jacobian"):
        ref = oracle.assemble(form, w.mesh, 2, fields=w.fields, constants=w.constants, cells=sample)
        for prec in ("fp64", "fp32", "bf16x3"):
            out = cf.coffee_assemble(form, 3, 2, coords, c2v, coeffs=dfs, constants=w.constants, precision=prec)
            torch.cuda.synchronize()
            got = out[idx].cpu().numpy()
            err = cell_rel_err(got.reshape(len(sample), -1), ref.reshape(len(sample), -1))
            print(f"svk_p2_tet full {form} {prec}: {err:.3e}")
            assert err < TOL[prec]
            del out


@pytest.mark.parametrize("d,p", [(3, 2), (3, 1), (2, 2)])
def test_svk_jacobian_ragged_counts(cf, oracle, d, p):
    """Cell counts that leave the last group of a wave partly empty (and a
    single cell), with the displacement given through a dof map and cell-major."""
    from gpu_util import TOL, assemble_gpu, cell_rel_err
    rng = np.random.default_rng(70 + 10 * d + p)
    mesh = I.make_mesh(d, 9 if d == 2 else 4, 0.1, rng)
    u = _disp(mesh, p, rng)
    ucm = I.Field(np.ascontiguousarray(u.values[u.cell_to_dof]), None, u.degree, u.ncomp)
    cst = [1.1, 0.9]
    for count in (1, 4, 5, 6, 11, 37):
        sub = I.Mesh(mesh.d, mesh.n, mesh.coords, np.ascontiguousarray(mesh.cells[:count]))
        ref = oracle.assemble("svk_jacobian", mesh, p, fields=[u], constants=cst, cells=np.arange(count))
        mapped = I.Field(u.values, np.ascontiguousarray(u.cell_to_dof[:count]), u.degree, u.ncomp)
        cellmajor = I.Field(np.ascontiguousarray(ucm.values[:count]), None, u.degree, u.ncomp)
        for f in (mapped, cellmajor):
            got = assemble_gpu("svk_jacobian", sub, p, [f], constants=cst, precision="fp64").cpu().numpy()
            err = cell_rel_err(got.reshape(count, -1), ref.reshape(count, -1))
            assert err < TOL["fp64"], (count, f.cell_to_dof is None, err)


def test_svk_energy_adjoint_full_size_sampled(cf, oracle):
    """196,608-cell SVK P2 tetrahedra: the energy's reverse pass over the whole
    mesh. The gradient at sampled vertices and displacement dofs equals the
    oracle's complex-step adjoint over the cells touching them; the whole
    coordinate gradient is translation invariant; the displacement gradient
    equals the assembled residual (R = dPi/du) scattered to the dofs."""
    import torch
    from gpu_util import to_dev
    w = I.workload("svk_p2_tet")
    mesh, u = w.mesh, w.fields[0]
    coords, c2v, dfs = to_dev(mesh, w.fields)
    cv = torch.empty(mesh.ncells, dtype=torch.float64, device=coords.device)
    gc, gu = cf.coffee_assemble_adjoint("svk_energy", 3, 2, coords, c2v, coeffs=dfs, constants=w.constants,
                                        seed=1.0, cell_value=cv)
    res = cf.coffee_assemble("svk_residual", 3, 2, coords, c2v, coeffs=dfs, constants=w.constants)
    torch.cuda.synchronize()
    # residual [E, 3 * 10] (component-blocked) scattered to [ndofs, 3]
    scat = torch.zeros_like(dfs[0].values)
    rb = res.reshape(mesh.ncells, 3, 10).permute(0, 2, 1).reshape(-1, 3)
    scat.index_add_(0, dfs[0].cell_to_dof.reshape(-1).long(), rb)
    gc, gu, scat = gc.cpu().numpy(), gu[0].cpu().numpy(), scat.cpu().numpy()
    assert np.max(np.abs(gu - scat)) < 1e-11 * np.max(np.abs(scat))
    scale = np.max(np.abs(gc))
    assert np.max(np.abs(gc.sum(axis=0))) < 1e-10 * scale * np.sqrt(mesh.nvert)
    rng = np.random.default_rng(21)
    for v in rng.integers(0, mesh.nvert, 5):
        cells = np.nonzero(np.any(mesh.cells == v, axis=1))[0]
        sub = I.Mesh(3, mesh.n, mesh.coords, mesh.cells[cells])
        f = I.Field(u.values, u.cell_to_dof[cells], 2, 3)
        _, gref, _ = oracle.adjoint("svk_energy", sub, 2, fields=[f], constants=w.constants)
        np.testing.assert_allclose(gc[v], gref[v], rtol=1e-9, atol=1e-10 * np.max(np.abs(gref[v])))
    for r in rng.integers(0, u.values.shape[0], 5):
        cells = np.nonzero(np.any(u.cell_to_dof == r, axis=1))[0]
        if cells.size == 0:
            continue
        sub = I.Mesh(3, mesh.n, mesh.coords, mesh.cells[cells])
        f = I.Field(u.values, u.cell_to_dof[cells], 2, 3)
        _, _, fref = oracle.adjoint("svk_energy", sub, 2, fields=[f], constants=w.constants)
        np.testing.assert_allclose(gu[r], fref[0][r], rtol=1e-9, atol=1e-10 * np.max(np.abs(fref[0][r])))


@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 2)])
@pytest.mark.parametrize("det", [False, True])
def test_svk_residual_adjoint(cf, oracle, d, p, det):
    """Reverse pass of S = sum_e lam_e^T b_e against the oracle's complex-step
    gradient; the displacement gradient also equals sum_e A_e lam_e with A_e
    the GPU Jacobian (the residual's derivative), scattered to the dofs."""
    import torch
    from gpu_util import to_dev
    rng = np.random.default_rng(80 + 10 * d + p)
    mesh = I.make_mesh(d, 6 if d == 2 else 3, 0.1, rng)
    u = _disp(mesh, p, rng)
    cst = [1.2, 0.8]
    N = oracle.tensor_dim("svk_residual", d, p)
    lam = rng.standard_normal((mesh.ncells, N))
    S_ref, gc_ref, gu_ref = oracle.adjoint("svk_residual", mesh, p, fields=[u], constants=cst, lam=lam)
    coords, c2v, dfs = to_dev(mesh, [u])
    lam_d = torch.as_tensor(lam, device=coords.device)
    cv = torch.empty(mesh.ncells, dtype=torch.float64, device=coords.device)
    gc, gu = cf.coffee_assemble_adjoint("svk_residual", d, p, coords, c2v, coeffs=dfs, constants=cst, lam=lam_d,
                                        cell_value=cv, deterministic=det)
    A = cf.coffee_assemble("svk_jacobian", d, p, coords, c2v, coeffs=dfs, constants=cst)
    torch.cuda.synchronize()
    rel = lambda a, b: float(np.max(np.abs(a - b)) / np.max(np.abs(b)))
    S = float(cv.sum())
    assert abs(S - S_ref) < 1e-11 * abs(S_ref)
    assert rel(gc.cpu().numpy(), gc_ref) < 1e-10
    assert rel(gu[0].cpu().numpy(), gu_ref[0]) < 1e-10
    ns = I.n_scalar_dofs(d, p)
    Al = torch.bmm(A, lam_d.unsqueeze(2)).reshape(mesh.ncells, d, ns).permute(0, 2, 1).reshape(-1, d)
    scat = torch.zeros_like(dfs[0].values).index_add_(0, dfs[0].cell_to_dof.reshape(-1).long(), Al)
    assert rel(gu[0].cpu().numpy(), scat.cpu().numpy()) < 1e-12


def test_svk_energy_deterministic(cf):
    """Energy reverse pass in deterministic mode on the full 196,608-cell P2
    workload: bitwise repeatable, equal to the atomic scatter to rounding."""
    import torch
    from gpu_util import to_dev
    w = I.workload("svk_p2_tet")
    coords, c2v, dfs = to_dev(w.mesh, w.fields)
    res = []
    for det in (True, True, False):
        gc, gu = cf.coffee_assemble_adjoint("svk_energy", 3, 2, coords, c2v, coeffs=dfs, constants=w.constants,
                                            deterministic=det)
        torch.cuda.synchronize()
        res.append((gc, gu[0]))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    for k in range(2):
        assert float((res[0][k] - res[2][k]).abs().max()) <= 1e-12 * float(res[2][k].abs().max())


def test_autograd_energy_and_residual_action(cf):
    """EnergyFn: gradients of Pi through torch.autograd equal the reverse pass,
    dPi/du matches central differences of the GPU energy, and without
    requires_grad the forward value is the same. ResidualActionFn likewise."""
    import torch
    from gpu_util import to_dev
    from paper_1407_0904_amd.autograd import svk_energy, svk_residual_action
    rng = np.random.default_rng(4)
    mesh = I.make_mesh(3, 3, 0.1, rng)
    u = _disp(mesh, 2, rng)
    cst = [1.0, 1.0]
    coords, c2v, dfs = to_dev(mesh, [u])
    Pi0 = svk_energy(3, 2, coords, c2v, dfs[0], constants=cst)
    coords.requires_grad_(True)
    dfs[0].values.requires_grad_(True)
    Pi = svk_energy(3, 2, coords, c2v, dfs[0], constants=cst)
    Pi.backward()
    gc, gu = cf.coffee_assemble_adjoint("svk_energy", 3, 2, coords.detach(), c2v,
                                        coeffs=[cf.DeviceField(dfs[0].values.detach(), dfs[0].cell_to_dof, 2, 3)],
                                        constants=cst)
    torch.cuda.synchronize()
    assert abs(float(Pi0) - float(Pi.detach())) <= 1e-14 * abs(float(Pi0))
    assert torch.allclose(coords.grad, gc, rtol=1e-13, atol=1e-16)
    assert torch.allclose(dfs[0].values.grad, gu[0], rtol=1e-13, atol=1e-16)

    def energy_at(vals):
        f = cf.DeviceField(vals, dfs[0].cell_to_dof, 2, 3)
        return float(cf.coffee_assemble("svk_energy", 3, 2, coords.detach(), c2v, coeffs=[f], constants=cst).sum())

    h = 1e-6
    for (r, c) in ((5, 0), (40, 2)):
        vp = dfs[0].values.detach().clone(); vp[r, c] += h
        vm = dfs[0].values.detach().clone(); vm[r, c] -= h
        fd = (energy_at(vp) - energy_at(vm)) / (2 * h)
        g = float(dfs[0].values.grad[r, c])
        assert abs(fd - g) <= 1e-6 * max(abs(fd), 1e-8)
    lam = torch.as_tensor(rng.standard_normal((mesh.ncells, 30)), device=coords.device)
    coords.grad = None
    dfs[0].values.grad = None
    S = svk_residual_action(3, 2, coords, c2v, dfs[0], lam, constants=cst)
    S.backward()
    gc2, gu2 = cf.coffee_assemble_adjoint("svk_residual", 3, 2, coords.detach(), c2v,
                                          coeffs=[cf.DeviceField(dfs[0].values.detach(), dfs[0].cell_to_dof, 2, 3)],
                                          constants=cst, lam=lam)
    torch.cuda.synchronize()
    assert torch.allclose(coords.grad, gc2, rtol=1e-13, atol=1e-16)
    assert torch.allclose(dfs[0].values.grad, gu2[0], rtol=1e-13, atol=1e-16)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 1), (2, 2)])
def test_svk_energy_residual_ragged_counts(cf, oracle, d, p, prec):
    """Energy and residual at counts around the 64-cell wave and the 256-cell workgroup, through a dof map and
    cell-major."""
    from gpu_util import TOL, assemble_gpu, cell_rel_err
    rng = np.random.default_rng(190 + 10 * d + p)
    mesh = I.make_mesh(d, 13 if d == 2 else 4, 0.1, rng)
    u = _disp(mesh, p, rng)
    cst = [1.2, 0.8]
    for count in (1, 63, 64, 65, 257):
        sub = I.Mesh(mesh.d, mesh.n, mesh.coords, np.ascontiguousarray(mesh.cells[:count]))
        mapped = I.Field(u.values, np.ascontiguousarray(u.cell_to_dof[:count]), u.degree, u.ncomp)
        cellmajor = I.Field(np.ascontiguousarray(u.values[mapped.cell_to_dof]), None, u.degree, u.ncomp)
        for form in ("svk_energy", "svk_residual"):
            ref = oracle.assemble(form, sub, p, fields=[mapped], constants=cst).reshape(count, -1)
            for f in (mapped, cellmajor):
                got = assemble_gpu(form, sub, p, [f], constants=cst, precision=prec).cpu().numpy().reshape(count, -1)
                assert cell_rel_err(got, ref) < TOL[prec], (form, count, f.cell_to_dof is None)


@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 1), (2, 2)])
def test_svk_energy_gradients_scattered_cells(cf, oracle, d, p):
    """Both gradients with the cells in random order (more distinct dofs per wave than the combining tables hold) and
    in mesh order, at counts around the wave and the workgroup, against the oracle's complex-step gradient."""
    import torch
    from gpu_util import to_dev
    rng = np.random.default_rng(290 + 10 * d + p)
    mesh = I.make_mesh(d, 17 if d == 2 else 5, 0.1, rng)
    u = _disp(mesh, p, rng)
    cst = [1.2, 0.8]
    for order in (np.arange(mesh.ncells), rng.permutation(mesh.ncells)):
        for count in (1, 65, 257, mesh.ncells):
            sub = I.Mesh(d, mesh.n, mesh.coords, np.ascontiguousarray(mesh.cells[order[:count]]))
            f = I.Field(u.values, np.ascontiguousarray(u.cell_to_dof[order[:count]]), u.degree, u.ncomp)
            S, gc, gu = oracle.adjoint("svk_energy", sub, p, fields=[f], constants=cst)
            coords, c2v, dfs = to_dev(sub, [f])
            cv = torch.empty(count, dtype=torch.float64, device=coords.device)
            hc, hu = cf.coffee_assemble_adjoint("svk_energy", d, p, coords, c2v, coeffs=dfs, constants=cst,
                                                cell_value=cv)
            for a, b in ((hc.cpu().numpy(), gc), (hu[0].cpu().numpy(), gu[0])):
                assert np.abs(a - b).max() <= 1e-11 * np.abs(b).max(), count
            assert abs(float(cv.sum()) - float(np.sum(S))) <= 1e-11 * abs(float(np.sum(S)))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 2)])
def test_svk_jacobian_counts_around_groups(cf, oracle, d, p, prec):
    """Jacobian at counts around the five-cell group and the twenty cells of a workgroup, through a dof map and
    cell-major, with large displacements (every term of the tangent matters)."""
    from gpu_util import TOL, assemble_gpu, cell_rel_err
    rng = np.random.default_rng(390 + 10 * d + p)
    mesh = I.make_mesh(d, 9 if d == 2 else 4, 0.1, rng)
    u = _disp(mesh, p, rng, sigma=0.2)
    cst = [1.2, 0.8]
    for count in (1, 4, 5, 6, 19, 20, 21, 101):
        sub = I.Mesh(mesh.d, mesh.n, mesh.coords, np.ascontiguousarray(mesh.cells[:count]))
        mapped = I.Field(u.values, np.ascontiguousarray(u.cell_to_dof[:count]), u.degree, u.ncomp)
        cellmajor = I.Field(np.ascontiguousarray(u.values[mapped.cell_to_dof]), None, u.degree, u.ncomp)
        ref = oracle.assemble("svk_jacobian", sub, p, fields=[mapped], constants=cst)
        for f in (mapped, cellmajor):
            got = assemble_gpu("svk_jacobian", sub, p, [f], constants=cst, precision=prec).cpu().numpy()
            assert cell_rel_err(got, ref) < TOL[prec], (count, f.cell_to_dof is None)


@pytest.mark.parametrize("d,p,n,fit,extra", [(3, 2, 23, 1, 65), (3, 1, 28, 2, 1), (2, 2, 320, 3, 127)])
def test_svk_energy_gradients_several_units_per_wave(cf, d, p, n, fit, extra):
    """More cells than one pass of the grid takes, with a ragged end: the per-cell energies equal those of calls on
    parts that one pass takes bit for bit, the gradients their sum (atomic order: 1e-12 of the largest)."""
    import torch
    from gpu_util import to_dev
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(11 + d + p)
    mesh = I.make_mesh(d, n, 0.1, rng)
    count = min(256 * cu * fit + extra, mesh.ncells)
    sub = I.Mesh(d, mesh.n, mesh.coords, np.ascontiguousarray(mesh.cells[:count]))
    coords, c2v, _ = to_dev(sub, [])
    dev, ns = c2v.device, I.n_scalar_dofs(d, p)
    ndofs = count * ns // 5 + ns
    dofs = (torch.arange(count * ns, device=dev) % ndofs).to(torch.int32).reshape(count, ns)
    vals = torch.as_tensor(0.05 * rng.standard_normal((ndofs, d)), device=dev)

    def call(a, b):
        u = cf.DeviceField(vals, dofs[a:b].contiguous(), p, d)
        e = torch.empty(b - a, dtype=torch.float64, device=dev)
        g, h = cf.coffee_assemble_adjoint("svk_energy", d, p, coords, c2v[a:b].contiguous(), coeffs=[u],
                                          constants=(1.0, 2.0), cell_value=e)
        return e, g, h[0]

    whole, half = call(0, count), count // 2
    lo, hi = call(0, half), call(half, count)
    assert torch.equal(whole[0], torch.cat((lo[0], hi[0])))
    for w, x, y in zip(whole[1:], lo[1:], hi[1:]):
        assert float((w - x - y).abs().max()) <= 1e-12 * float(w.abs().max())


@pytest.mark.parametrize("cellmajor", [True, False])
@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 1), (2, 2)])
def test_svk_residual_adjoint_without_displacement_gradient(cf, d, p, cellmajor):
    """The residual's reverse pass with the displacement gradient skipped (values alone; coordinates alone), with more
    distinct dofs per wave than a combining table holds: what is left equals the full pass."""
    import torch
    from gpu_util import to_dev
    rng = np.random.default_rng(490 + 10 * d + p)
    mesh = I.make_mesh(d, 17 if d == 2 else 5, 0.1, rng)
    count, ns = 257, I.n_scalar_dofs(d, p)
    sub = I.Mesh(d, mesh.n, mesh.coords, np.ascontiguousarray(mesh.cells[rng.permutation(mesh.ncells)[:count]]))
    coords, c2v, _ = to_dev(sub, [])
    dev = coords.device
    vals = torch.as_tensor(rng.normal(0, 0.05, (count * ns, d)), device=dev)
    dofs = torch.as_tensor(rng.permutation(count * ns).astype(np.int32).reshape(count, ns), device=dev)
    u = cf.DeviceField(vals[dofs.long()].contiguous() if cellmajor else vals, None if cellmajor else dofs, p, d)
    lam = torch.as_tensor(rng.standard_normal((count, d * ns)), device=dev)
    cv = [torch.empty(count, dtype=torch.float64, device=dev) for _ in range(3)]
    full, _ = cf.coffee_assemble_adjoint("svk_residual", d, p, coords, c2v, coeffs=[u], lam=lam, cell_value=cv[0])
    cf.coffee_assemble_adjoint("svk_residual", d, p, coords, c2v, coeffs=[u], lam=lam, cell_value=cv[1], grads=False)
    only, _ = cf.coffee_assemble_adjoint("svk_residual", d, p, coords, c2v, coeffs=[u], lam=lam, cell_value=cv[2],
                                         grad_coeffs=[None])
    torch.cuda.synchronize()
    assert torch.equal(cv[0], cv[1]) and torch.equal(cv[0], cv[2])
    assert float((full - only).abs().max()) <= 1e-12 * float(full.abs().max())


@pytest.mark.parametrize("cellmajor", [True, False])
@pytest.mark.parametrize("d,p", [(3, 1), (3, 2), (2, 1), (2, 2)])
def test_svk_energy_values_alone(cf, oracle, d, p, cellmajor):
    """The energy's reverse pass without any gradient array runs the forward kernel: its values against the oracle, at
    counts around a wave and a workgroup; nothing beyond them is written, and no values at all is a call that succeeds."""
    import torch
    from gpu_util import TOL, cell_rel_err, to_dev
    rng = np.random.default_rng(510 + 10 * d + p)
    mesh = I.make_mesh(d, 17 if d == 2 else 5, 0.1, rng)
    u = _disp(mesh, p, rng)
    cst = [1.3, 0.7]
    ref = oracle.assemble("svk_energy", mesh, p, fields=[u], constants=cst).reshape(-1, 1)
    coords, c2v, _ = to_dev(mesh, [])
    dev = coords.device
    vals, dofs = torch.as_tensor(u.values, device=dev), torch.as_tensor(u.cell_to_dof, device=dev)
    for count in (1, 63, 64, 65, 257, 514):
        m = dofs[:count].contiguous()
        f = cf.DeviceField(vals[m.long()].contiguous() if cellmajor else vals, None if cellmajor else m, p, d)
        cv = torch.full((count + 1,), -7.0, dtype=torch.float64, device=dev)
        args = ("svk_energy", d, p, coords, c2v[:count].contiguous())
        cf.coffee_assemble_adjoint(*args, coeffs=[f], constants=cst, cell_value=cv[:count], grads=False)
        cf.coffee_assemble_adjoint(*args, coeffs=[f], constants=cst, grads=False)
        got = cv.cpu().numpy()
        assert cell_rel_err(got[:count].reshape(-1, 1), ref[:count]) < TOL["fp64"] and got[count] == -7.0
