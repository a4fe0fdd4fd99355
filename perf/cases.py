"""Performance cases of the library: the assemblies a finite element program asks for.

Each case is one call (or one differentiable evaluation) through the public
Python entry points on a synthetic jittered mesh held on the GPU, in the tuned
launch configuration the package ships. `listed()` names the standing cases,
`draw()` gives more of the same ranges, `prepare()` builds what a program
holds before the call (mesh, dof maps, coefficients, output buffers, CSR
pattern, batch descriptors), `run()` is one pass, `work()` counts the bytes and
operations the pass cannot do without, and `exact()` evaluates the same
quadrature sums in plain FP64 torch (rules, bases and integrands written here,
independently of the library).

Meshes: unit square or cube, n per side, split into triangles, Kuhn tetrahedra
or extruded triangle prisms (numbered column by column), interior vertices
jittered; `cells` keeps the first cells of the mesh, as one part of a
partition does, so that counts are not multiples of any tile.
"""
import math
import os
from itertools import permutations

import numpy as np
import torch

from paper_1407_0904_amd import autograd, coffee

_CODE = {"triangle": 2, "tetrahedron": 3, "prism": 6}
_TRI_EDGES = ((1, 2), (0, 2), (0, 1))
_TET_EDGES = ((2, 3), (1, 3), (1, 2), (0, 3), (0, 2), (0, 1))
_VECTOR = ("elasticity", "burgers", "svk_energy", "svk_residual", "svk_jacobian")
_TUNING = os.path.join(os.path.dirname(os.path.abspath(coffee.__file__)), "tuning_mi355x.txt")
_MAX_OUT = 3_000_000_000  # bytes of output of a drawn case

coffee.coffee_load_tuning(_TUNING)


def _case(name, call, form, cell, degree, field_degree, precision, n, cells=None, **more):
    c = {"call": call, "form": form, "cell": cell, "degree": degree, "field_degree": field_degree,
         "precision": precision, "n": n, "cells": _mesh_cells(cell, n) if cells is None else cells, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one time step of a small 2-D problem: the call's latency is what counts
        _case("helmholtz_p1_tri_8k", "assemble", "helmholtz", "triangle", 1, 1, "fp64", 64),
        # a large 2-D mesh at the lowest degree (one part of a partition: an odd cell count)
        _case("helmholtz_p1_tri_2m", "assemble", "helmholtz", "triangle", 1, 1, "fp64", 1021, 2_084_881),
        # the benchmark's headline workload: reaction-diffusion operator, P2 tetrahedra, P2 coefficient
        _case("helmholtz_p2_tet", "assemble", "helmholtz", "tetrahedron", 2, 2, "fp64", 64),
        # the same operator summed into a CSR matrix whose pattern the program keeps
        _case("helmholtz_p2_tet_csr", "csr", "helmholtz", "tetrahedron", 2, 1, "fp64", 40),
        # stiffness blocks of linear elasticity with varying Lame parameters
        _case("elasticity_p2_tet", "assemble", "elasticity", "tetrahedron", 2, 1, "fp64", 48),
        # shape and parameter sensitivities of an elastic functional: forward and backward
        _case("elasticity_p2_tet_grad", "gradient", "elasticity", "tetrahedron", 2, 1, "fp64", 48,
              deterministic=False),
        # Newton matrix of a viscous Burgers time step
        _case("burgers_p2_tet", "assemble", "burgers", "tetrahedron", 2, 2, "fp64", 48),
        # Newton matrix of a hyperelastic solid
        _case("svk_jacobian_p2_tet", "assemble", "svk_jacobian", "tetrahedron", 2, 2, "fp64", 32),
        # energy minimisation of the same solid: energy and its gradients, forward and backward
        _case("svk_energy_p2_tet_grad", "gradient", "svk_energy", "tetrahedron", 2, 2, "fp64", 32,
              deterministic=False),
        # extruded (ocean, atmosphere) meshes: diffusion on prisms
        _case("diffusion_p2_prism", "assemble", "diffusion", "prism", 2, 0, "fp64", 64),
        # the same at higher degree in split-bf16 precision, an odd cell count
        _case("diffusion_p3_prism_bf16x3", "assemble", "diffusion", "prism", 3, 0, "bf16x3", 32, 65_497),
        # hp-adaptive serving batch: 3,000,000 cells of mixed shape, degree and form in random order
        {"name": "mixed_batch_3m", "call": "batch", "entries": 3_000_000, "precision": "fp32", "layout": "packed",
         "n_tri": 1000, "n_tet": 56},
    ]


def draw(rng):
    call = rng.choices(["assemble", "gradient", "csr", "batch"], weights=[12, 3, 2, 2])[0]
    prec = rng.choices(["fp64", "fp32", "bf16x3"], weights=[5, 3, 2])[0]
    if call == "batch":
        entries = int(round(math.exp(rng.uniform(math.log(3_000), math.log(3_000_000)))))
        n_tri = max(4, math.ceil(math.sqrt(entries / 3.0)))            # 2 n^2 triangles for 2/3 of the entries
        n_tet = max(2, math.ceil((entries / 18.0) ** (1 / 3)))         # 6 n^3 tetrahedra for 1/3
        return {"call": "batch", "entries": entries, "precision": "fp32" if prec == "bf16x3" else prec,
                "layout": rng.choice(["packed", "caller"]), "n_tri": n_tri, "n_tet": n_tet}
    if call == "csr":
        form = rng.choice(["mass", "helmholtz", "elasticity"])
        cell = rng.choice(["triangle", "tetrahedron"])
        p, fd = rng.choice([1, 2]), 1
        prec = "fp32" if prec == "bf16x3" else prec
        most = 40_000_000 // _dim(form, cell, p) ** 2
        return _case(None, "csr", form, cell, p, fd, prec, _side(cell, _spread(rng, 2_000, most)))
    if call == "gradient":
        form = rng.choice(["helmholtz", "elasticity", "svk_energy"])
        cell = rng.choice(["triangle", "tetrahedron", "tetrahedron"])
        p = rng.choice([1, 2, 2])
        # the coefficient in the trial space where the reverse pass is compiled for that, else P1
        fd = p if form == "svk_energy" or (form == "helmholtz" and cell == "tetrahedron") else 1
        most = 600_000 if form == "elasticity" else 200_000
        cells = _spread(rng, 2_000, most)
        return _case(None, "gradient", form, cell, p, fd, "fp64", _side(cell, cells), cells,
                     deterministic=rng.random() < 0.2)
    form = rng.choice(["mass", "helmholtz", "helmholtz", "diffusion", "elasticity", "elasticity", "burgers",
                       "burgers", "svk_jacobian", "svk_residual", "svk_energy"])
    if form in ("mass", "helmholtz", "diffusion"):
        cell = rng.choice(["triangle", "tetrahedron", "prism"])
        p = rng.choice([1, 2, 3])
        fd = 0 if form == "diffusion" else rng.choice([0, 1] if cell == "prism" else [0, 1, 2])
    else:
        cell = rng.choice(["triangle", "tetrahedron", "tetrahedron"])
        p = rng.choice([1, 2, 2])
        fd = rng.choice([0, 1, 1]) if form == "elasticity" else p
    most = min(2_000_000, _MAX_OUT // (_out_values(form, cell, p) * (8 if prec == "fp64" else 4)))
    if cell == "prism":
        most = min(most, 500_000 if p < 3 else 65_000)
    elif form.startswith("svk"):
        most = min(most, 200_000)
    cells = _spread(rng, 1_000, most)
    return _case(None, "assemble", form, cell, p, fd, prec, _side(cell, cells), cells)


def _spread(rng, least, most):
    return int(round(math.exp(rng.uniform(math.log(least), math.log(most)))))


# ---------------------------------------------------------------- sizes

def _mesh_cells(cell, n):
    return 2 * n * n if cell == "triangle" else 6 * n ** 3 if cell == "tetrahedron" else 2 * n ** 3


def _side(cell, cells):
    n = 2
    while _mesh_cells(cell, n) < cells:
        n += 1
    return n


def _gdim(cell):
    return 2 if cell == "triangle" else 3


def _nscalar(cell, p):
    if cell == "prism":
        return (p + 1) * (p + 2) // 2 * (p + 1)
    return (p + 1) * (p + 2) // 2 if cell == "triangle" else (p + 1) * (p + 2) * (p + 3) // 6


def _dim(form, cell, p):
    return _nscalar(cell, p) * (_gdim(cell) if form in _VECTOR else 1)


def _out_values(form, cell, p):
    n = _dim(form, cell, p)
    return 1 if form == "svk_energy" else n if form == "svk_residual" else n * n


# ---------------------------------------------------------------- meshes (torch, on the device)

def _lattice(m, d, dev):
    """Integer lattice points [m^d, d], first axis fastest."""
    i = torch.arange(m ** d, device=dev)
    return torch.stack([(i // m ** a) % m for a in range(d)], dim=1)


def _square(n, dev):
    s = torch.arange(n * n, device=dev)
    a = (s % n) + (s // n) * (n + 1)
    b, c, d = a + 1, a + n + 1, a + n + 2
    return torch.stack([torch.stack([a, b, d], 1), torch.stack([a, d, c], 1)], 1).reshape(-1, 3)


def _cube(n, dev):
    s = torch.arange(n ** 3, device=dev)
    m = n + 1
    base = (s % n) + ((s // n) % n) * m + (s // (n * n)) * m * m
    step = (1, m, m * m)
    tets = []
    for perm in permutations(range(3)):
        p1 = step[perm[0]]
        verts = [0, p1, p1 + step[perm[1]], sum(step)]
        if sum(perm[x] > perm[y] for x in range(3) for y in range(x + 1, 3)) % 2:
            verts[2], verts[3] = verts[3], verts[2]
        tets.append(torch.stack([base + v for v in verts], 1))
    return torch.stack(tets, 1).reshape(-1, 4)


def _prisms(n, dev):
    m = n + 1
    bot = _square(n, dev)[:, None, :] * m + torch.arange(n, device=dev)[None, :, None]
    return torch.stack([bot[..., 0], bot[..., 0] + 1, bot[..., 1], bot[..., 1] + 1, bot[..., 2], bot[..., 2] + 1],
                       -1).reshape(-1, 6)


def _mesh(cell, n, gen, dev):
    """(coords [V, d] float64, cells [E, nv] int64), interior vertices jittered."""
    d = _gdim(cell)
    lat = _lattice(n + 1, d, dev)
    r = 0.20 if cell == "triangle" else 0.10
    shift = (torch.rand(lat.shape, generator=gen, device=dev, dtype=torch.float64) * 2 - 1) * (r / n)
    shift[((lat == 0) | (lat == n)).any(1)] = 0.0
    coords = lat.double() / n + shift
    if cell != "prism":
        return coords, (_square if cell == "triangle" else _cube)(n, dev)
    m = n + 1
    v = torch.arange(m ** 3, device=dev)            # vertex b m + k is lattice point b + m^2 k
    return coords[(v // m) + m * m * (v % m)].contiguous(), _prisms(n, dev)


def _p2_map(cells, n, d, dev):
    """Degree-2 dofs of simplices: the points of the twice-refined lattice."""
    lat, mr = _lattice(n + 1, d, dev), 2 * n + 1
    w = torch.tensor([mr ** a for a in range(d)], device=dev)
    at = (lat * w).sum(1)[cells]                    # index contribution of each vertex
    cols = [2 * at[:, a] for a in range(d + 1)]
    cols += [at[:, a] + at[:, b] for a, b in (_TRI_EDGES if d == 2 else _TET_EDGES)]
    return torch.stack(cols, 1).to(torch.int32).contiguous(), mr ** d


def _fields(case, c2v, nvert, n, gen, dev):
    """Coefficient fields with the distributions the forms meet in use."""
    form, fd, d = case["form"], case["field_degree"], _gdim(case["cell"])
    if fd == 0:
        return []
    ncomp = d if form in ("burgers", "svk_energy", "svk_residual", "svk_jacobian") else 1
    if fd == 1:
        cmap, nd = c2v, nvert
    else:
        cmap, nd = _p2_map(c2v.long(), n, d, dev)
    lo, hi = {"elasticity": (1.0, 10.0), "burgers": (-1.0, 1.0)}.get(form, (0.5, 1.5))
    out = []
    for _ in range(2 if form == "elasticity" else 1):
        if form.startswith("svk"):
            v = torch.randn((nd, ncomp), generator=gen, device=dev, dtype=torch.float64) * 0.01
        else:
            v = torch.rand((nd, ncomp), generator=gen, device=dev, dtype=torch.float64) * (hi - lo) + lo
        out.append(coffee.DeviceField(v, cmap, fd, ncomp))
    return out


def _constants(case):
    form = case["form"]
    if form == "elasticity":
        return [] if case["field_degree"] else [1.0, 2.0]
    return [1.0, 1.0] if form in ("burgers", "diffusion") or form.startswith("svk") else []


# ---------------------------------------------------------------- prepare and run

_BINS = [("triangle", p, c) for p, c in ((1, 800), (2, 600), (3, 400), (4, 200))] + \
        [("tetrahedron", p, c) for p, c in ((1, 500), (2, 300), (3, 200))]


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _prepare_batch(case, gen, dev):
    meshes, pools = {}, {}
    for cell, n in (("triangle", case["n_tri"]), ("tetrahedron", case["n_tet"])):
        x, c = _mesh(cell, n, gen, dev)
        c = c.to(torch.int32).contiguous()
        f = torch.rand((x.shape[0], 1), generator=gen, device=dev, dtype=torch.float64) + 0.5
        meshes[cell] = (x, c, coffee.DeviceField(f, c, 1, 1))
        pools[cell] = torch.randperm(c.shape[0], generator=gen, device=dev)
    # bins: (form, cell, degree), the costliest (largest tensors) first
    bins = sorted(((f, c, p) for c, p, _ in _BINS for f in ("mass", "helmholtz")), key=lambda b: -_nscalar(b[1], b[2]))
    at = {b: i for i, b in enumerate(bins)}
    segs = [coffee.Segment(f, _CODE[c], p, *meshes[c]) for f, c, p in bins]
    seg_of, cell_of = [], []
    taken, left = {"triangle": 0, "tetrahedron": 0}, case["entries"]
    for i, (cell, p, share) in enumerate(_BINS):
        k = left if i == len(_BINS) - 1 else case["entries"] * share // 3000
        k = min(k, pools[cell].shape[0] - taken[cell])
        left -= k
        ids = pools[cell][taken[cell]:taken[cell] + k]
        taken[cell] += k
        helm = torch.randint(0, 2, (k,), generator=gen, device=dev)
        seg_of.append(torch.where(helm == 1, at[("helmholtz", cell, p)], at[("mass", cell, p)]))
        cell_of.append(ids)
    seg_of, cell_of = torch.cat(seg_of), torch.cat(cell_of)
    perm = torch.randperm(seg_of.shape[0], generator=gen, device=dev)
    seg_of, cell_of = seg_of[perm].to(torch.int32).contiguous(), cell_of[perm].contiguous()
    size = torch.tensor([_nscalar(c, p) ** 2 for _, c, p in bins], device=dev)[seg_of.long()]
    total = int(size.sum())
    odt = torch.float64 if case["precision"] == "fp64" else torch.float32
    ent = seg_of.shape[0]
    st = {"call": "batch", "packed": case["layout"] == "packed", "segs": segs, "bins": bins, "seg_of": seg_of,
          "cell_of": cell_of, "total": total, "precision": case["precision"],
          "out": torch.empty(total, dtype=odt, device=dev),
          "offset": torch.cumsum(size, 0) - size,
          "workspace": torch.empty(coffee.coffee_batch_workspace_size(len(segs), ent), dtype=torch.uint8, device=dev)}
    if st["packed"]:
        st["offset"] = torch.empty(ent, dtype=torch.int64, device=dev)
    return st


def _problem(case, seed):
    """Mesh, fields and vectors of a case, from the seed alone."""
    dev = _dev()
    gen = torch.Generator(device=dev).manual_seed(seed)
    coords, cells = _mesh(case["cell"], case["n"], gen, dev)
    c2v = cells[:case["cells"]].to(torch.int32).contiguous()
    fields = _fields(case, c2v, coords.shape[0], case["n"], gen, dev)
    lam = u = None
    if case["call"] == "gradient" and case["form"] != "svk_energy":
        shape = (c2v.shape[0], _dim(case["form"], case["cell"], case["degree"]))
        lam = torch.randn(shape, generator=gen, device=dev, dtype=torch.float64)
        u = torch.randn(shape, generator=gen, device=dev, dtype=torch.float64)
    return coords, c2v, fields, lam, u


def prepare(case, seed):
    dev = _dev()
    if case["call"] == "batch":
        return _prepare_batch(case, torch.Generator(device=dev).manual_seed(seed), dev)
    coords, c2v, fields, lam, u = _problem(case, seed)
    st = {"call": case["call"], "form": case["form"], "code": _CODE[case["cell"]], "degree": case["degree"],
          "precision": case["precision"], "coords": coords, "c2v": c2v, "fields": fields,
          "constants": _constants(case)}
    odt = torch.float64 if case["precision"] == "fp64" else torch.float32
    if case["call"] == "assemble":
        shape = coffee.output_shape(case["form"], c2v.shape[0], st["code"], case["degree"])
        st["out"] = torch.empty(shape, dtype=odt, device=dev)
    elif case["call"] == "gradient":
        st["deterministic"] = case["deterministic"]
        st["lam"], st["u"] = lam, u
        coords.requires_grad_(True)
        for f in fields:
            f.values.requires_grad_(True)
    else:  # csr: the pattern belongs to the mesh, the program keeps it
        d = _gdim(case["cell"])
        dofs, nd = (c2v, coords.shape[0]) if case["degree"] == 1 else _p2_map(c2v.long(), case["n"], d, dev)
        ncomp = d if case["form"] in _VECTOR else 1
        st["dofs"], st["ndofs"] = dofs, nd
        st["row_ptr"], st["col_idx"] = coffee.coffee_csr_pattern(dofs, nd, ncomp)
        st["values"] = torch.empty(st["col_idx"].numel(), dtype=odt, device=dev)
    return st


def run(s):
    if s["call"] == "assemble":
        return coffee.coffee_assemble(s["form"], s["code"], s["degree"], s["coords"], s["c2v"], coeffs=s["fields"],
                                      constants=s["constants"], precision=s["precision"], out=s["out"])
    if s["call"] == "gradient":
        wrt = [s["coords"]] + [f.values for f in s["fields"]]
        if s["form"] == "svk_energy":
            S = autograd.svk_energy(s["code"], s["degree"], s["coords"], s["c2v"], s["fields"][0],
                                    constants=s["constants"], deterministic=s["deterministic"])
        else:
            S = autograd.bilinear_action(s["form"], s["code"], s["degree"], s["coords"], s["c2v"],
                                         fields=s["fields"], constants=s["constants"], lam=s["lam"], u=s["u"],
                                         deterministic=s["deterministic"])
        return [S.detach(), *torch.autograd.grad(S, wrt)]
    if s["call"] == "csr":
        return coffee.coffee_assemble_csr(s["form"], s["code"], s["degree"], s["coords"], s["c2v"], s["row_ptr"],
                                          s["col_idx"], s["ndofs"], cell_to_dof=s["dofs"], coeffs=s["fields"],
                                          constants=s["constants"], precision=s["precision"], values=s["values"])
    if s["packed"]:
        return coffee.coffee_assemble_batch_packed(s["segs"], s["seg_of"], s["cell_of"], s["total"],
                                                   precision=s["precision"], out=s["out"], out_offset=s["offset"],
                                                   workspace=s["workspace"])
    return coffee.coffee_assemble_batch(s["segs"], s["seg_of"], s["cell_of"], s["offset"], s["total"],
                                        precision=s["precision"], out=s["out"], workspace=s["workspace"])


# ---------------------------------------------------------------- work

def _mesh_bytes(cell, n, cells, field_degree=0, ncomp=1, nfield=1):
    d = _gdim(cell)
    nv = {"triangle": 3, "tetrahedron": 4, "prism": 6}[cell]
    part = cells / _mesh_cells(cell, n)
    b = part * (n + 1) ** d * d * 8 + cells * nv * 4
    if field_degree == 1:
        b += part * (n + 1) ** d * ncomp * nfield * 8
    elif field_degree == 2:
        b += part * (2 * n + 1) ** d * ncomp * nfield * 8 + cells * _nscalar(cell, 2) * 4
    return b


def work(case):
    """Each input read once, each output written once; per cell the geometry
    (about 60 operations, at every point on prisms, whose map is not affine)
    and d + 1 multiply-adds for each distinct value."""
    if case["call"] == "batch":
        out = flops = ent = 0.0
        for cell, p, share in _BINS:
            k = case["entries"] * share / 3000
            ns, d = _nscalar(cell, p), _gdim(cell)
            ent, out = ent + k, out + k * ns * ns
            flops += k * (60 + (d + 1) * ns * (ns + 1))
        mesh = sum(_mesh_bytes(c, n, min(_mesh_cells(c, n), case["entries"] * s), 1)
                   for c, n, s in (("triangle", case["n_tri"], 2 / 3), ("tetrahedron", case["n_tet"], 1 / 3)))
        return {"bytes": mesh + ent * (4 + 8 + 8) + out * (8 if case["precision"] == "fp64" else 4), "flops": flops}
    form, cell, p, cells = case["form"], case["cell"], case["degree"], case["cells"]
    d, dim = _gdim(cell), _dim(form, cell, p)
    ncomp = d if form in _VECTOR and form != "elasticity" else 1
    nfield = 2 if form == "elasticity" else 1
    item = 8 if case["precision"] == "fp64" else 4
    inp = _mesh_bytes(cell, case["n"], cells, case["field_degree"], ncomp, nfield)
    vals = _out_values(form, cell, p)
    distinct = vals if form in ("burgers", "svk_residual", "svk_energy") else dim * (dim + 1) // 2
    points = 1 if cell != "prism" else (p + 1) ** 3
    flops = cells * (60 * points + 2 * (d + 1) * distinct)
    if case["call"] == "assemble":
        return {"bytes": inp + cells * vals * item, "flops": flops}
    if case["call"] == "gradient":
        # inputs and their gradients, lam and u; the gradients at the points take as much again as the values
        vec = 0 if form == "svk_energy" else 2 * cells * dim * 8
        maps = cells * 4 * ((3 if cell == "triangle" else 4) + (_nscalar(cell, 2) if case["field_degree"] == 2 else 0))
        return {"bytes": inp + (inp - maps) + vec, "flops": cells * (180 + 12 * (d + 1) * dim)}
    # csr: the dof map and the pattern are read, the values written; neighbours per dof from the lattice
    per_row = {("triangle", 1): 7, ("triangle", 2): 11.5, ("tetrahedron", 1): 15, ("tetrahedron", 2): 28}[cell, p]
    nd = (case["n"] * p + 1) ** d
    nc = d if form in _VECTOR else 1
    dofmap = cells * 4 * _nscalar(cell, p) if p == 2 else 0
    return {"bytes": inp + dofmap + nd * nc * 8 + nd * per_row * nc * nc * (4 + item), "flops": flops}


# ---------------------------------------------------------------- the same sums in plain FP64

def _gauss_jacobi(m, alpha):
    """m-point rule on [0, 1] for the weight (1 - x)^alpha (Golub-Welsch)."""
    k = np.arange(m, dtype=np.float64)
    s = 2 * k + alpha
    diag = np.where(k == 0, -alpha / (alpha + 2.0), -alpha ** 2 / np.maximum(s * (s + 2), 1e-300))
    j = np.arange(1, m, dtype=np.float64)
    t = 2 * j + alpha
    off = np.sqrt(4 * j * (j + alpha) * j * (j + alpha) / (t * t * (t + 1) * (t - 1)))
    x, v = np.linalg.eigh(np.diag(diag) + np.diag(off, 1) + np.diag(off, -1))
    return (1 + x) / 2, v[0] ** 2 / (alpha + 1)


def _rule(cell, q):
    """Collapsed Gauss-Jacobi product rule of degree q (prisms: triangle rule times Gauss-Legendre)."""
    m = (q + 2) // 2
    x0, w0 = _gauss_jacobi(m, 0)
    x1, w1 = _gauss_jacobi(m, 1)
    if cell == "tetrahedron":
        x2, w2 = _gauss_jacobi(m, 2)
        return [((a, (1 - a) * b, (1 - a) * (1 - b) * c), wa * wb * wc)
                for a, wa in zip(x2, w2) for b, wb in zip(x1, w1) for c, wc in zip(x0, w0)]
    tri = [((a, (1 - a) * b), wa * wb) for a, wa in zip(x1, w1) for b, wb in zip(x0, w0)]
    if cell == "triangle":
        return tri
    return [((*x, z), w * wz) for x, w in tri for z, wz in zip(x0, w0)]


def _nodes(d, p):
    """Barycentric lattice indices of the degree-p simplex nodes, in dof order."""
    def unit(*pairs):
        a = [0] * (d + 1)
        for i, k in pairs:
            a[i] += k
        return tuple(a)
    out = [unit((v, p)) for v in range(d + 1)]
    for a, b in (_TRI_EDGES if d == 2 else _TET_EDGES):
        out += [unit((a, p - k), (b, k)) for k in range(1, p)]
    faces = [(0, 1, 2)] if d == 2 else [tuple(v for v in range(4) if v != f) for f in range(4)]
    for f in faces:
        out += [unit((f[0], p - i - j), (f[1], i), (f[2], j)) for j in range(1, p) for i in range(1, p - j)]
    if d == 3:
        out += [(p - i - j - k, i, j, k) for k in range(1, p) for j in range(1, p - k) for i in range(1, p - j - k)]
    return out


def _simplex_basis(d, p, X):
    """Lagrange values [n] and reference gradients [n, d] at X, as products of linear factors."""
    bary = [1.0 - sum(X), *X]
    dbary = [[-1.0] * d] + [[1.0 if i == j else 0.0 for j in range(d)] for i in range(d)]
    val, grad = [], []
    for al in _nodes(d, p):
        f, df = [], []
        for i, k in enumerate(al):      # prod_{l<k} (p lambda_i - l) / (l + 1) and its derivative in lambda_i
            fac = [(p * bary[i] - l) / (l + 1) for l in range(k)]
            f.append(math.prod(fac))
            df.append(sum(p / (l + 1) * math.prod(fac[:l] + fac[l + 1:]) for l in range(k)))
        val.append(math.prod(f))
        grad.append([sum(df[i] * dbary[i][j] * math.prod(f[:i] + f[i + 1:]) for i in range(d + 1)) for j in range(d)])
    return val, grad


def _interval_basis(p, z):
    nodes = [0.0, 1.0] + [k / p for k in range(1, p)]
    val, der = [], []
    for b, xb in enumerate(nodes):
        fac = [((z - x) / (xb - x), 1.0 / (xb - x)) for c, x in enumerate(nodes) if c != b]
        val.append(math.prod(f for f, _ in fac))
        der.append(sum(fac[i][1] * math.prod(f for j, (f, _) in enumerate(fac) if j != i) for i in range(len(fac))))
    return val, der


def _basis(cell, p, X, dev):
    if cell != "prism":
        v, g = _simplex_basis(_gdim(cell), p, X)
    else:
        tv, tg = _simplex_basis(2, p, X[:2])
        lv, lg = _interval_basis(p, X[2])
        v = [a * b for a in tv for b in lv]
        g = [[ga[0] * b, ga[1] * b, a * gb] for a, ga in zip(tv, tg) for b, gb in zip(lv, lg)]
    return torch.tensor(v, dtype=torch.float64, device=dev), torch.tensor(g, dtype=torch.float64, device=dev)


def _geometry(x, G1):
    """K = J^-1 and |det J| from vertex positions x [E, nv, d] and vertex-basis gradients G1 [nv, d]."""
    J = torch.matmul(x.transpose(1, 2).contiguous(), G1)
    c = lambda i, j: J[:, i, j]  # noqa: E731
    if J.shape[1] == 2:
        det = c(0, 0) * c(1, 1) - c(0, 1) * c(1, 0)
        adj = torch.stack([c(1, 1), -c(0, 1), -c(1, 0), c(0, 0)], 1).reshape(-1, 2, 2)
    else:
        co = lambda i, j: (c((i + 1) % 3, (j + 1) % 3) * c((i + 2) % 3, (j + 2) % 3)  # noqa: E731
                           - c((i + 1) % 3, (j + 2) % 3) * c((i + 2) % 3, (j + 1) % 3))
        det = c(0, 0) * co(0, 0) + c(0, 1) * co(0, 1) + c(0, 2) * co(0, 2)
        adj = torch.stack([co(j, i) for i in range(3) for j in range(3)], 1).reshape(-1, 3, 3)
    return adj / det[:, None, None], det.abs()


def _points(case, x, quad):
    """Per point: weight |det J| [E], basis values [n] and physical gradients [E, n, d] of the space, K."""
    dev, cell = x.device, case["cell"]
    K = None
    for X, w in _rule(cell, quad):
        if K is None or cell == "prism":
            K, det = _geometry(x, _basis(cell, 1, X, dev)[1])
        phi, dphi = _basis(cell, case["degree"], X, dev)
        yield X, w * det, phi, torch.matmul(dphi, K), K


def _at(case, X, K, loc):
    """A field with local dofs loc [E, nloc, ncomp] at X: values [E, ncomp], gradients [E, ncomp, d]."""
    phi, dphi = _basis(case["cell"], case["field_degree"], X, loc.device)
    lt = loc.transpose(1, 2).contiguous()
    return torch.matmul(lt, phi), torch.matmul(torch.matmul(lt, dphi), K)


def _svk(case, X, K, loc):
    mu, lm = _constants(case)
    H = _at(case, X, K, loc)[1]
    eye = torch.eye(H.shape[1], dtype=H.dtype, device=H.device)
    F = eye + H
    E = 0.5 * (H + H.transpose(1, 2) + torch.matmul(H.transpose(1, 2).contiguous(), H))
    tr = E.diagonal(dim1=1, dim2=2).sum(1)
    S = lm * tr[:, None, None] * eye + 2 * mu * E
    psi = 0.5 * lm * tr * tr + mu * (E * E).sum((1, 2))
    return F, S, psi, mu, lm


def _tensors(case, x, locs):
    """Element tensors of the cells with vertices x [E, nv, d] and local field dofs locs."""
    form, p, cell = case["form"], case["degree"], case["cell"]
    E, d, ns = x.shape[0], x.shape[2], _nscalar(cell, p)
    quad = 2 * p + 1 if form == "burgers" else 2 * p
    vec = form in _VECTOR
    out = torch.zeros((E, d, ns, d, ns) if vec else (E, ns, ns), dtype=torch.float64, device=x.device)
    if form == "svk_energy":
        out = torch.zeros(E, dtype=torch.float64, device=x.device)
    elif form == "svk_residual":
        out = torch.zeros((E, d, ns), dtype=torch.float64, device=x.device)
    cst = _constants(case)
    for X, wd, phi, g, K in _points(case, x, quad):
        wg = wd[:, None, None] * g
        gt = g.transpose(1, 2).contiguous()
        if form in ("mass", "helmholtz", "diffusion"):
            if form != "mass":
                out += torch.matmul(wg if form == "helmholtz" else cst[0] * cst[1] * wg, gt)
            if form != "diffusion":
                f = _at(case, X, K, locs[0])[0][:, 0] if locs else 1.0
                out += (wd * f)[:, None, None] * torch.outer(phi, phi)
        elif form == "elasticity":
            mu, lm = ([_at(case, X, K, v)[0][:, 0] for v in locs] if locs
                      else [torch.full_like(wd, c) for c in cst])
            full = torch.matmul(wg, gt)
            for c in range(d):
                out[:, c, :, c, :] += mu[:, None, None] * full
                for e in range(d):
                    out[:, c, :, e, :] += wg[:, :, e, None] * g[:, None, :, c] * mu[:, None, None] \
                        + wg[:, :, c, None] * g[:, None, :, e] * lm[:, None, None]
        elif form == "burgers":
            w, dw = _at(case, X, K, locs[0])
            conv = torch.matmul(g, w[:, :, None])[:, :, 0]
            same = cst[0] * torch.matmul(wg, gt) \
                + wd[:, None, None] * (cst[1] * torch.outer(phi, phi) + phi[:, None] * conv[:, None, :])
            pp = torch.outer(phi, phi)
            for c in range(d):
                out[:, c, :, c, :] += same
                for e in range(d):
                    out[:, c, :, e, :] += (wd * dw[:, c, e])[:, None, None] * pp
        else:
            F, S, psi, mu, lm = _svk(case, X, K, locs[0])
            if form == "svk_energy":
                out += wd * psi
            elif form == "svk_residual":
                out += torch.matmul(torch.matmul(F, S), (wd[:, None, None] * gt))
            else:
                FF = torch.matmul(F, F.transpose(1, 2).contiguous())
                Fg = torch.matmul(F, gt)                       # [E, c, a] = sum_j F_cj g_aj
                gg = torch.matmul(g, gt)
                geo = torch.matmul(torch.matmul(g, S), gt)
                for c in range(d):
                    out[:, c, :, c, :] += wd[:, None, None] * geo
                    for e in range(d):
                        out[:, c, :, e, :] += wd[:, None, None] * (
                            lm * Fg[:, c, :, None] * Fg[:, e, None, :] + mu * Fg[:, e, :, None] * Fg[:, c, None, :]
                            + mu * FF[:, c, e, None, None] * gg)
    return out if not vec or form.startswith("svk_energy") else out.reshape(
        (E, d * ns) if form == "svk_residual" else (E, d * ns, d * ns))


def _functional(case, x, locs, lam, u):
    """Sum over the cells of lam^T A u, or of the energy."""
    total = 0.0
    d, p = x.shape[2], case["degree"]
    for X, wd, phi, g, K in _points(case, x, 2 * p):
        if case["form"] == "svk_energy":
            total = total + (wd * _svk(case, X, K, locs[0])[2]).sum()
            continue
        vals = [_at(case, X, K, v)[0][:, 0] for v in locs]
        if case["form"] == "helmholtz":
            gl, gu = torch.matmul(lam[:, None, :], g), torch.matmul(u[:, None, :], g)
            total = total + (wd * ((gl * gu).sum((1, 2)) + vals[0] * (lam @ phi) * (u @ phi))).sum()
        else:
            L = torch.matmul(lam.reshape(-1, d, lam.shape[1] // d), g)
            U = torch.matmul(u.reshape(-1, d, u.shape[1] // d), g)
            el, eu = 0.5 * (L + L.transpose(1, 2)), 0.5 * (U + U.transpose(1, 2))
            tl, tu = (v.diagonal(dim1=1, dim2=2).sum(1) for v in (L, U))
            total = total + (wd * (2 * vals[0] * (el * eu).sum((1, 2)) + vals[1] * tl * tu)).sum()
    return total


def _chunks(count, per_cell):
    step = max(1, min(count, 200_000_000 // max(per_cell, 1)))
    return [(i, min(count, i + step)) for i in range(0, count, step)]


def _all_tensors(case, coords, c2v, fields):
    return torch.cat([_tensors(case, coords[c2v[i:j].long()], [f.values[f.cell_to_dof[i:j].long()] for f in fields])
                      for i, j in _chunks(c2v.shape[0], 3 * _out_values(case["form"], case["cell"], case["degree"]))])


def exact(case, seed):
    if case["call"] == "batch":
        s = prepare(case, seed)
        out = torch.empty(s["total"], dtype=torch.float64, device=s["out"].device)
        off = s["offset"].clone()
        seg = s["seg_of"].long()
        at = 0
        for b, (form, cell, p) in enumerate(s["bins"]):
            sub = {"form": form, "cell": cell, "degree": p, "field_degree": 1}
            idx = torch.nonzero(seg == b)[:, 0]
            nn = _nscalar(cell, p) ** 2
            if s["packed"]:     # segment by segment, entries in input order
                off[idx] = at + nn * torch.arange(idx.shape[0], device=off.device)
                at += nn * idx.shape[0]
            sg = s["segs"][b]
            for i, j in _chunks(idx.shape[0], 3 * nn):
                rows = s["cell_of"][idx[i:j]]
                v = sg.cell_to_vertex[rows].long()
                A = _tensors(sub, sg.coords[v], [sg.coeff.values[v]])
                out[off[idx[i:j]][:, None] + torch.arange(nn, device=off.device)] = A.reshape(j - i, nn)
        return (out, off) if s["packed"] else out
    coords, c2v, fields, lam, u = _problem(case, seed)
    if case["call"] == "assemble":
        return _all_tensors(case, coords, c2v, fields)
    if case["call"] == "gradient":
        wrt = [coords.requires_grad_(True)] + [f.values.requires_grad_(True) for f in fields]
        total, grads = 0.0, [torch.zeros_like(v) for v in wrt]
        for i, j in _chunks(c2v.shape[0], 2000):
            S = _functional(case, coords[c2v[i:j].long()], [f.values[f.cell_to_dof[i:j].long()] for f in fields],
                            None if lam is None else lam[i:j], None if u is None else u[i:j])
            for a, b in zip(grads, torch.autograd.grad(S, wrt)):
                a += b
            total = total + S.detach()
        return [total, *grads]
    # csr: entry (row, column) of each pair of dofs found among the pattern's sorted keys
    s = prepare(case, seed)
    nc = s["row_ptr"].shape[0] // s["ndofs"]
    rows = torch.repeat_interleave(torch.arange(s["row_ptr"].shape[0] - 1, device=coords.device),
                                   s["row_ptr"][1:] - s["row_ptr"][:-1])
    keys = rows * (s["ndofs"] * nc) + s["col_idx"]
    vals = torch.zeros(keys.shape[0], dtype=torch.float64, device=coords.device)
    for i, j in _chunks(c2v.shape[0], 4 * _out_values(case["form"], case["cell"], case["degree"])):
        A = _tensors(case, coords[c2v[i:j].long()], [f.values[f.cell_to_dof[i:j].long()] for f in fields])
        g = torch.cat([s["dofs"][i:j].long() * nc + c for c in range(nc)], 1)
        vals.index_add_(0, torch.searchsorted(keys, (g[:, :, None] * (s["ndofs"] * nc) + g[:, None, :]).reshape(-1)),
                        A.reshape(-1))
    return vals
