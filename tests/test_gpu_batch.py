"""GPU mixed persistent batch (coffee_assemble_batch): equal to per-bin
launches bit for bit, equal to the oracle within the precision's bar."""
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


def device_batch(cf, mb, variant=0, task_cells=0, order=None):
    import torch
    dev = torch.device("cuda:0")
    tri_c = torch.as_tensor(mb.tri.coords, device=dev)
    tri_v = torch.as_tensor(mb.tri.cells, device=dev)
    tet_c = torch.as_tensor(mb.tet.coords, device=dev)
    tet_v = torch.as_tensor(mb.tet.cells, device=dev)
    f_tri = cf.DeviceField.from_host(mb.f_tri, dev)
    f_tet = cf.DeviceField.from_host(mb.f_tet, dev)
    segs = []
    for (form, d, p) in mb.segments:
        c, v, f = (tri_c, tri_v, f_tri) if d == 2 else (tet_c, tet_v, f_tet)
        vv = variant[len(segs)] if isinstance(variant, (list, tuple)) else variant
        segs.append(cf.Segment(form, d, p, c, v, f, variant=vv, task_cells=task_cells))
    arrays = (torch.as_tensor(mb.seg_of, device=dev), torch.as_tensor(mb.cell_of, device=dev),
              torch.as_tensor(mb.out_offset, device=dev))
    return segs, arrays


def per_bin_reference(cf, mb, segs, precision):
    """Per-bin coffee_assemble launches, scattered into batch order on the host."""
    import torch
    out = np.zeros(mb.total_elems, dtype=np.float64 if precision == "fp64" else np.float32)
    for b, (form, d, p) in enumerate(mb.segments):
        idx = np.nonzero(mb.seg_of == b)[0]
        if idx.size == 0:
            continue
        sg = segs[b]
        cells = torch.as_tensor(mb.cell_of[idx], device=sg.coords.device)
        sub_c2v = sg.cell_to_vertex[cells].contiguous()
        sub_f = cf.DeviceField(sg.coeff.values, sg.coeff.cell_to_dof[cells].contiguous(), 1, 1)
        A = cf.coffee_assemble(form, d, p, sg.coords, sub_c2v, coeffs=[sub_f], precision=precision)
        A = A.reshape(idx.size, -1).cpu().numpy()
        nn = A.shape[1]
        for k, i in enumerate(idx):
            o = mb.out_offset[i]
            out[o:o + nn] = A[k]
    return out


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("variant,task_cells", [(0, 64), (1, 64), (0, 256), (1, 128), (0, 1024), (1, 512)])
def test_batch_equals_per_bin_launches(cf, precision, variant, task_cells):
    import torch
    mb = I.mixed_batch(n_tri=24, n_tet=6, tri_counts=(400, 300, 200, 100), tet_counts=(500, 300, 200), seed=7)
    segs, (seg_of, cell_of, offs) = device_batch(cf, mb, variant, task_cells)
    got = cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, precision=precision)
    torch.cuda.synchronize()
    ref = per_bin_reference(cf, mb, segs, precision)
    np.testing.assert_array_equal(got.cpu().numpy(), ref)


def test_batch_vs_oracle(cf, oracle):
    import torch
    from gpu_util import TOL
    mb = I.mixed_batch(n_tri=16, n_tet=4, tri_counts=(200, 150, 100, 50), tet_counts=(150, 100, 80), seed=3)
    segs, (seg_of, cell_of, offs) = device_batch(cf, mb, variant=[b % 2 for b in range(14)], task_cells=128)
    got = cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, precision="fp32").cpu().numpy()
    worst = 0.0
    for b, (form, d, p) in enumerate(mb.segments):
        idx = np.nonzero(mb.seg_of == b)[0]
        mesh, f = (mb.tri, mb.f_tri) if d == 2 else (mb.tet, mb.f_tet)
        ref = oracle.assemble(form, mesh, p, fields=[f], cells=mb.cell_of[idx])
        nn = ref.shape[1] * ref.shape[2]
        g = np.stack([got[mb.out_offset[i]:mb.out_offset[i] + nn] for i in idx]).astype(np.float64)
        r = ref.reshape(len(idx), -1)
        err = np.max(np.max(np.abs(g - r), 1) / np.max(np.abs(r), 1))
        worst = max(worst, err)
    print(f"batch vs oracle worst cell rel err {worst:.3e}")
    assert worst < TOL["fp32"]


def test_batch_full_size_sampled(cf):
    """The 3,000,000-entry mixed batch: sampled entries equal per-bin launches bit for bit."""
    import torch
    mb = I.mixed_batch()
    segs, (seg_of, cell_of, offs) = device_batch(cf, mb)
    got = cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, precision="fp32")
    torch.cuda.synchronize()
    rng = np.random.default_rng(0)
    for b, (form, d, p) in enumerate(mb.segments):
        idx = np.nonzero(mb.seg_of == b)[0]
        pick = np.sort(rng.choice(idx, size=min(200, idx.size), replace=False))
        sg = segs[b]
        cells = torch.as_tensor(mb.cell_of[pick], device=sg.coords.device)
        sub_f = cf.DeviceField(sg.coeff.values, sg.coeff.cell_to_dof[cells].contiguous(), 1, 1)
        A = cf.coffee_assemble(form, d, p, sg.coords, sg.cell_to_vertex[cells].contiguous(), coeffs=[sub_f],
                               precision="fp32").reshape(len(pick), -1)
        nn = A.shape[1]
        gidx = torch.as_tensor((mb.out_offset[pick][:, None] + np.arange(nn)[None, :]).reshape(-1), device=got.device)
        np.testing.assert_array_equal(got[gidx].reshape(len(pick), nn).cpu().numpy(), A.cpu().numpy())


def test_batch_full_size_vs_oracle(cf, oracle):
    """The 3,000,000-entry mixed batch in the tuned launch shape the benchmark
    times (both layouts): sampled entries of every bin against the oracle."""
    import os
    import torch
    from gpu_util import TOL
    tuning = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1407_0904_amd",
                          "tuning_mi355x.txt")
    cf.coffee_load_tuning(tuning)
    try:
        mb = I.mixed_batch()
        segs, (seg_of, cell_of, offs) = device_batch(cf, mb)
        got = cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, precision="fp32")
        gotp, poff = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, mb.total_elems, precision="fp32")
        torch.cuda.synchronize()
        poff = poff.cpu().numpy()
        rng = np.random.default_rng(9)
        worst = 0.0
        for b, (form, d, p) in enumerate(mb.segments):
            idx = np.nonzero(mb.seg_of == b)[0]
            pick = np.sort(rng.choice(idx, size=min(150, idx.size), replace=False))
            mesh, f = (mb.tri, mb.f_tri) if d == 2 else (mb.tet, mb.f_tet)
            ref = oracle.assemble(form, mesh, p, fields=[f], cells=mb.cell_of[pick]).reshape(len(pick), -1)
            nn = ref.shape[1]
            for out, offsets in ((got, mb.out_offset), (gotp, poff)):
                gidx = torch.as_tensor((offsets[pick][:, None] + np.arange(nn)[None, :]).reshape(-1),
                                       device=out.device)
                g = out[gidx].reshape(len(pick), nn).cpu().numpy().astype(np.float64)
                err = float(np.max(np.max(np.abs(g - ref), 1) / np.max(np.abs(ref), 1)))
                worst = max(worst, err)
                assert err < TOL["fp32"], (form, d, p, err)
        print(f"3M batch vs oracle, worst sampled cell rel err {worst:.3e}")
    finally:
        cf.coffee_load_tuning(None)


def test_batch_validation(cf):
    import torch
    mb = I.mixed_batch(n_tri=4, n_tet=2, tri_counts=(4, 4, 4, 4), tet_counts=(4, 4, 4), seed=2)
    segs, (seg_of, cell_of, offs) = device_batch(cf, mb)
    with pytest.raises(cf.CoffeeError) as ei:
        cf.coffee_assemble_batch(segs[:0], seg_of, cell_of, offs, mb.total_elems)
    assert ei.value.code == 1
    bad = list(segs)
    bad[0] = cf.Segment("elasticity", 2, 1, segs[0].coords, segs[0].cell_to_vertex, segs[0].coeff)
    with pytest.raises(cf.CoffeeError) as ei:
        cf.coffee_assemble_batch(bad, seg_of, cell_of, offs, mb.total_elems)
    assert ei.value.code == 2
    bad[0] = cf.Segment("mass", 2, 1, segs[0].coords, segs[0].cell_to_vertex, segs[0].coeff, task_cells=100)
    with pytest.raises(cf.CoffeeError) as ei:
        cf.coffee_assemble_batch(bad, seg_of, cell_of, offs, mb.total_elems)
    assert ei.value.code == 1
    small = torch.empty(16, dtype=torch.uint8, device=seg_of.device)
    with pytest.raises(ValueError, match="workspace has"):
        cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, workspace=small)


@pytest.mark.parametrize("packed", [False, True])
def test_batch_skips_out_of_range_entries(cf, packed):
    """Entries whose segment id is outside [0, nseg) or whose cell index is
    outside the segment's mesh are skipped: nothing is written for them (the
    packed layout returns offset -1), and every other entry is unchanged."""
    import torch
    mb = I.mixed_batch(n_tri=8, n_tet=3, tri_counts=(40, 30, 20, 10), tet_counts=(30, 20, 10), seed=5)
    segs, (seg_of, cell_of, offs) = device_batch(cf, mb, 0, 64)
    n = seg_of.shape[0]
    bad = np.array([3, 17, 40, 41, n - 1])
    so = mb.seg_of.copy()
    co = mb.cell_of.copy()
    so[3], so[17] = -1, len(mb.segments)          # segment id out of range
    co[40], co[41], co[n - 1] = -5, 10 ** 9, -1   # cell index out of range
    seg_bad = torch.as_tensor(so, device=seg_of.device)
    cell_bad = torch.as_tensor(co, device=seg_of.device)
    keep = np.setdiff1d(np.arange(n), bad)
    if packed:
        ref, roff = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, mb.total_elems, precision="fp64")
        got, goff = cf.coffee_assemble_batch_packed(segs, seg_bad, cell_bad, mb.total_elems, precision="fp64")
        torch.cuda.synchronize()
        goff = goff.cpu().numpy()
        assert np.all(goff[bad] == -1)
        # the kept entries of each segment stay in input order, packed from the segment's start
        g, r, ro = got.cpu().numpy(), ref.cpu().numpy(), roff.cpu().numpy()
        nn = np.array([I.n_scalar_dofs(d, p) ** 2 for (_, d, p) in mb.segments])[mb.seg_of]
        for i in keep:
            np.testing.assert_array_equal(g[goff[i]:goff[i] + nn[i]], r[ro[i]:ro[i] + nn[i]])
    else:
        ref = cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, precision="fp64")
        out = torch.full((mb.total_elems,), 7.25, dtype=torch.float64, device=seg_of.device)
        got = cf.coffee_assemble_batch(segs, seg_bad, cell_bad, offs, mb.total_elems, precision="fp64", out=out)
        torch.cuda.synchronize()
        g, r = got.cpu().numpy(), ref.cpu().numpy()
        nn = np.array([I.n_scalar_dofs(d, p) ** 2 for (_, d, p) in mb.segments])[mb.seg_of]
        for i in bad:
            assert np.all(g[mb.out_offset[i]:mb.out_offset[i] + nn[i]] == 7.25)
        for i in keep:
            np.testing.assert_array_equal(g[mb.out_offset[i]:mb.out_offset[i] + nn[i]],
                                          r[mb.out_offset[i]:mb.out_offset[i] + nn[i]])


def packed_offsets(mb):
    """The packed layout from its definition: segments in order, each segment's
    entries in increasing entry index, tensors back to back."""
    nn = np.array([I.n_scalar_dofs(d, p) ** 2 for (_, d, p) in mb.segments], dtype=np.int64)
    off = np.empty(mb.seg_of.shape[0], dtype=np.int64)
    pos = 0
    for b in range(len(mb.segments)):
        idx = np.nonzero(mb.seg_of == b)[0]
        off[idx] = pos + nn[b] * np.arange(idx.size, dtype=np.int64)
        pos += nn[b] * idx.size
    return off, int(pos)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("task_cells", [64, 256, 1024])
def test_packed_batch_layout_and_values(cf, precision, task_cells):
    """coffee_assemble_batch_packed: the returned offsets are the packed layout
    exactly, every tensor equals the per-bin launch bit for bit, and a second
    call reproduces the offsets."""
    import torch
    mb = I.mixed_batch(n_tri=24, n_tet=6, tri_counts=(400, 300, 200, 100), tet_counts=(500, 300, 200), seed=7)
    segs, (seg_of, cell_of, _) = device_batch(cf, mb, 0, task_cells)
    exp_off, total = packed_offsets(mb)
    assert total == mb.total_elems
    got, off = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, total, precision=precision)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(off.cpu().numpy(), exp_off)
    ref_scattered = per_bin_reference(cf, mb, segs, precision)  # tensors at mb.out_offset
    nn = np.array([I.n_scalar_dofs(d, p) ** 2 for (_, d, p) in mb.segments], dtype=np.int64)[mb.seg_of]
    g = got.cpu().numpy()
    for i in range(0, mb.seg_of.shape[0], 7):
        np.testing.assert_array_equal(g[exp_off[i]:exp_off[i] + nn[i]],
                                      ref_scattered[mb.out_offset[i]:mb.out_offset[i] + nn[i]])
    _, off2 = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, total, precision=precision)
    np.testing.assert_array_equal(off2.cpu().numpy(), exp_off)


def test_packed_batch_edge_cases(cf, oracle):
    """One entry; segments with no entries; counts that are not multiples of a
    task or of 16; against the oracle."""
    import torch
    from gpu_util import TOL
    for counts in [((1, 0, 0, 0), (0, 0, 0)), ((0, 17, 0, 3), (0, 0, 33)), ((65, 1, 129, 15), (1, 64, 7))]:
        mb = I.mixed_batch(n_tri=12, n_tet=4, tri_counts=counts[0], tet_counts=counts[1], seed=11)
        segs, (seg_of, cell_of, _) = device_batch(cf, mb, 0, 64)
        exp_off, total = packed_offsets(mb)
        got, off = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, total, precision="fp32")
        torch.cuda.synchronize()
        np.testing.assert_array_equal(off.cpu().numpy(), exp_off)
        g = got.cpu().numpy()
        for b, (form, d, p) in enumerate(mb.segments):
            idx = np.nonzero(mb.seg_of == b)[0]
            if idx.size == 0:
                continue
            mesh, f = (mb.tri, mb.f_tri) if d == 2 else (mb.tet, mb.f_tet)
            ref = oracle.assemble(form, mesh, p, fields=[f], cells=mb.cell_of[idx]).reshape(idx.size, -1)
            gg = np.stack([g[exp_off[i]:exp_off[i] + ref.shape[1]] for i in idx]).astype(np.float64)
            err = np.max(np.max(np.abs(gg - ref), 1) / np.max(np.abs(ref), 1))
            assert err < TOL["fp32"], (counts, form, d, p, err)


def test_packed_batch_full_size_sampled(cf):
    """The 3,000,000-entry mixed batch in the packed layout: offsets equal the
    layout's definition; sampled entries equal per-bin launches bit for bit."""
    import torch
    mb = I.mixed_batch()
    segs, (seg_of, cell_of, _) = device_batch(cf, mb)
    exp_off, total = packed_offsets(mb)
    got, off = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, total, precision="fp32")
    torch.cuda.synchronize()
    np.testing.assert_array_equal(off.cpu().numpy(), exp_off)
    rng = np.random.default_rng(1)
    for b, (form, d, p) in enumerate(mb.segments):
        idx = np.nonzero(mb.seg_of == b)[0]
        pick = np.sort(rng.choice(idx, size=min(200, idx.size), replace=False))
        sg = segs[b]
        cells = torch.as_tensor(mb.cell_of[pick], device=sg.coords.device)
        sub_f = cf.DeviceField(sg.coeff.values, sg.coeff.cell_to_dof[cells].contiguous(), 1, 1)
        A = cf.coffee_assemble(form, d, p, sg.coords, sg.cell_to_vertex[cells].contiguous(), coeffs=[sub_f],
                               precision="fp32").reshape(len(pick), -1)
        nn = A.shape[1]
        gidx = torch.as_tensor((exp_off[pick][:, None] + np.arange(nn)[None, :]).reshape(-1), device=got.device)
        np.testing.assert_array_equal(got[gidx].reshape(len(pick), nn).cpu().numpy(), A.cpu().numpy())


@pytest.mark.parametrize("packed", [False, True])
def test_batch_cell_major_field(cf, packed):
    """A field given cell-major (no dof map) gives the same bits as the same
    values behind a dof map, in every bin, in both layouts."""
    import torch
    mb = I.mixed_batch(n_tri=16, n_tet=4, tri_counts=(150, 100, 80, 50), tet_counts=(120, 80, 60), seed=11)
    segs, (seg_of, cell_of, offs) = device_batch(cf, mb, variant=[b % 2 for b in range(14)], task_cells=128)
    cm = []
    for sg in segs:
        v = sg.coeff.values[sg.coeff.cell_to_dof.long()].contiguous()  # [E, nloc, 1]
        cm.append(cf.Segment(sg.form, sg.cell, sg.degree, sg.coords, sg.cell_to_vertex,
                             cf.DeviceField(v, None, 1, 1), variant=sg.variant, task_cells=sg.task_cells))
    if packed:
        a, oa = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, mb.total_elems, precision="fp64")
        b, ob = cf.coffee_assemble_batch_packed(cm, seg_of, cell_of, mb.total_elems, precision="fp64")
        assert torch.equal(oa, ob)
    else:
        a = cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, precision="fp64")
        b = cf.coffee_assemble_batch(cm, seg_of, cell_of, offs, mb.total_elems, precision="fp64")
    torch.cuda.synchronize()
    np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("entries", [14, 1400, 140_000, 560_000])
def test_batch_task_size_by_entries(cf, precision, entries):
    """Tasks sized by the number of entries (and the grid by the tasks): equal
    to tasks of a given size bit for bit, both layouts."""
    import torch
    k = entries // 14
    n_tri, n_tet = int((4 * k) ** 0.5) + 2, int(k ** (1 / 3)) + 2
    mb = I.mixed_batch(n_tri=n_tri, n_tet=n_tet, tri_counts=(2 * k,) * 4, tet_counts=(2 * k,) * 3, seed=entries)
    res = []
    for task_cells in (0, 1024):
        segs, (seg_of, cell_of, offs) = device_batch(cf, mb, 0, task_cells)
        got = cf.coffee_assemble_batch(segs, seg_of, cell_of, offs, mb.total_elems, precision=precision)
        gotp, poff = cf.coffee_assemble_batch_packed(segs, seg_of, cell_of, mb.total_elems, precision=precision)
        res.append((got.cpu().numpy(), gotp.cpu().numpy(), poff.cpu().numpy()))
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)
