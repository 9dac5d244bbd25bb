"""GPU parity of the smoothed-aggregation setup and of the operators the
V-cycle applies: aggregates equal the oracle's exactly; P, coarse operators,
spectral bounds, SpMV and the V-cycle agree to rounding."""
import numpy as np
import pytest

from oracle import amg, assembly
from synth import box_mesh, face_coeff, fl_planar_front
from tests.gpu_util import case, csr, gpu_solver, rel_max, to_dev

pytestmark = pytest.mark.gpu


def _cases():
    yield "c1", case()
    m = box_mesh((23, 19, 17), jitter=0.1, seed=4)
    f = fl_planar_front(m.cell_centre, seed=7)
    yield "ragged_front", (m, f, face_coeff(m, 2400.0), None)
    # a tall all-liquid box: level 2 holds an aggregate of more than 64
    # members, which the bookkeeping ranks with the whole wavefront
    m = box_mesh((32, 32, 96), jitter=0.1, seed=0)
    yield "tall", (m, np.ones(m.n_cells), face_coeff(m, 2400.0), None)


@pytest.mark.parametrize("name,cs", list(_cases()), ids=lambda x: x if isinstance(x, str) else "")
def test_hierarchy_matches_oracle(name, cs):
    m, f, c, _ = cs
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    H = amg.build_hierarchy(sy.A)
    if name == "tall":
        assert max(np.bincount(lev.agg[lev.agg >= 0]).max() for lev in H.levels[:-1]) > 64
    s = gpu_solver(m, f, c)
    assert s.n_levels() == len(H.levels)
    for lvl, lev in enumerate(H.levels):
        info = s.level_info(lvl)
        n = lev.A.shape[0]
        assert info["n"] == n
        if lev.Ainv is None:
            assert abs(info["rho"] - lev.rho) <= 1e-12 * lev.rho, (lvl, info["rho"], lev.rho)
        else:  # solved through its inverse: no smoother, no bound computed
            assert info["rho"] == 0.0
        A = csr(*s.level_matrix(lvl), (n, n))
        assert rel_max(A, lev.A) <= 1e-13, lvl
        if lvl < len(H.levels) - 1:
            agg = s.aggregates(lvl).cpu().numpy()
            assert np.array_equal(agg, lev.agg), lvl           # exact
            P = csr(*s.prolongator(lvl), lev.P.shape)
            assert rel_max(P, lev.P) <= 1e-13, lvl


def test_spmv_and_vcycle_match_oracle():
    import torch

    m, f, c, _ = case()
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    H = amg.build_hierarchy(sy.A)
    s = gpu_solver(m, f, c)
    rng = np.random.default_rng(3)
    for lvl, lev in enumerate(H.levels):
        x = rng.normal(size=lev.A.shape[0])
        y = s.apply_matrix(lvl, to_dev(x, torch.float64)).cpu().numpy()
        ref = lev.A @ x
        assert np.abs(y - ref).max() <= 1e-14 * np.abs(lev.A).max() * np.abs(x).sum() / len(x) * 50
    r = rng.normal(size=sy.n_active)
    z = s.apply_vcycle(to_dev(r, torch.float64)).cpu().numpy()
    zr = amg.vcycle(H, r)
    assert np.linalg.norm(z - zr) <= 1e-12 * np.linalg.norm(zr)


def test_setup_is_deterministic():
    m, f, c, _ = case(shape=(20, 20, 20), fl="front")
    s1 = gpu_solver(m, f, c)
    s2 = gpu_solver(m, f, c)
    for lvl in range(s1.n_levels()):
        for a, b in zip(s1.level_matrix(lvl), s2.level_matrix(lvl)):
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())


def _vcycle_case(name):
    if name.startswith("c1"):
        return case()
    if name == "cube22":
        m, f, c, _ = case(shape=(22, 22, 22), fl="front", fl_seed=2, seed=2)
        return m, f, c, None
    if name == "ragged_front":
        m = box_mesh((23, 19, 17), jitter=0.1, seed=4)
        return m, fl_planar_front(m.cell_centre, seed=7), face_coeff(m, 2400.0), None
    raise ValueError(name)


# The coarsest operator is inverted by one workgroup's 4 x 4-blocked
# Gauss-Jordan up to 128 rows and by the 32 x 32-blocked form over many
# workgroups above that (ragged last blocks included); coarse_max picks
# which one a hierarchy ends in, down to a single aggregate of one row.
@pytest.mark.parametrize("name,coarse_max,n_coarsest", [
    ("c1", 8, 1), ("cube22", 16, 2), ("c1", 128, 16), ("ragged_front", 128, 25),
    ("cube22", 128, 40), ("c1", 400, 279), ("ragged_front", 512, 466), ("cube22", 1024, 728)])
def test_coarsest_inverse_variants(name, coarse_max, n_coarsest):
    import torch

    m, f, c, _ = _vcycle_case(name)
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    H = amg.build_hierarchy(sy.A, coarse_max=coarse_max)
    if n_coarsest is not None:
        assert H.levels[-1].A.shape[0] == n_coarsest
    s = gpu_solver(m, f, c, coarse_max=coarse_max)
    assert s.n_levels() == len(H.levels)
    r = np.random.default_rng(5).normal(size=sy.n_active)
    z = s.apply_vcycle(to_dev(r, torch.float64)).cpu().numpy()
    zr = amg.vcycle(H, r)
    assert np.linalg.norm(z - zr) <= 1e-12 * np.linalg.norm(zr)


def test_full_size_64cube_hierarchy():
    """The 64^3 timestep the benchmark times first: every level's aggregates
    exactly, operators and prolongators to rounding, and one V-cycle."""
    import torch

    from synth import fl_growing_front

    m = box_mesh((64, 64, 64), lengths=(0.01,) * 3, jitter=0.1, seed=0)
    c = face_coeff(m, 2400.0)
    f = fl_growing_front(m.cell_centre, t=0.101, t_end=0.2, s_max=0.6, delta=0.1, axis=0,
                         length=0.01)
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    H = amg.build_hierarchy(sy.A)
    s = gpu_solver(m, f, c)
    assert s.n_levels() == len(H.levels)
    for lvl, lev in enumerate(H.levels):
        n = lev.A.shape[0]
        A = csr(*s.level_matrix(lvl), (n, n))
        assert rel_max(A, lev.A) <= 1e-13, lvl
        if lvl < len(H.levels) - 1:
            assert np.array_equal(s.aggregates(lvl).cpu().numpy(), lev.agg), lvl
            P = csr(*s.prolongator(lvl), lev.P.shape)
            assert rel_max(P, lev.P) <= 1e-13, lvl
    r = np.random.default_rng(6).normal(size=sy.n_active)
    z = s.apply_vcycle(to_dev(r, torch.float64)).cpu().numpy()
    assert np.linalg.norm(z - amg.vcycle(H, r)) <= 1e-12 * np.linalg.norm(z)


def test_hierarchy_on_a_graph_of_degree_ten():
    """Extra faces to the in-plane diagonal neighbours give rows of up to ten
    off-diagonal entries: the finest level's ELL strength, MIS-2 and joining
    passes take their plain slot loop (more than eight slots) and the finest
    products the general sparse product.  Aggregates equal the oracle's,
    operators and prolongators agree to rounding, and so does one V-cycle."""
    import torch

    import paper_1810_08572_amd as ppe

    m = box_mesh((10, 9, 8), jitter=0.1, seed=3)
    idx = {tuple(g): c for c, g in enumerate(m.grid_index)}
    extra = [(c, idx[(i + di, j + dj, k)]) for c, (i, j, k) in enumerate(m.grid_index)
             for di, dj in ((1, 1), (1, -1)) if (i + di, j + dj, k) in idx]
    extra = np.array(extra)
    owner = np.concatenate([m.owner, extra[:, 0]]).astype(np.int32)
    neigh = np.concatenate([m.neigh, extra[:, 1]]).astype(np.int32)
    c0 = face_coeff(m, 2400.0)
    c = np.concatenate([c0, np.full(len(extra), 0.3 * c0[m.neigh >= 0].mean())])
    f = np.clip((m.cell_centre[:, 0] - 0.2) / 0.5, 0.0, 1.0)
    inner = neigh >= 0
    deg = np.bincount(np.concatenate([owner[inner], neigh[inner]]), minlength=m.n_cells)
    assert deg.max() > 8
    sy = assembly.masked_system(m.n_cells, owner, neigh, c, f)
    H = amg.build_hierarchy(sy.A, coarse_max=32)
    assert len(H.levels) >= 3
    s = ppe.Solver(coarse_max=32)
    s.set_mesh(m.n_cells, to_dev(owner, torch.int32), to_dev(neigh, torch.int32))
    s.assemble(to_dev(c, torch.float64), to_dev(f, torch.float64))
    assert s.n_levels() == len(H.levels)
    for lvl, lev in enumerate(H.levels):
        n = lev.A.shape[0]
        A = csr(*s.level_matrix(lvl), (n, n))
        assert A.nnz == lev.A.nnz and rel_max(A, lev.A) <= 1e-13, lvl
        if lvl < len(H.levels) - 1:
            assert np.array_equal(s.aggregates(lvl).cpu().numpy(), lev.agg), lvl
            P = csr(*s.prolongator(lvl), lev.P.shape)
            assert rel_max(P, lev.P) <= 1e-13, lvl
    r = np.random.default_rng(11).normal(size=sy.n_active)
    z = s.apply_vcycle(to_dev(r, torch.float64)).cpu().numpy()
    assert np.linalg.norm(z - amg.vcycle(H, r)) <= 1e-12 * np.linalg.norm(z)
    s.close()


@pytest.mark.parametrize("shape,links", [((60, 50, 1), 0), ((24, 20, 10), 4), ((24, 20, 10), 9),
                                         ((24, 20, 10), 120), ((24, 20, 10), 1500)])
def test_products_with_one_long_row(shape, links):
    """A cell weakly joined to cells all over the mesh: its row of A P has one
    column per aggregate it reaches.  A plane and four links are the edges of
    the finest level's passes on rows of up to four and eight entries, nine
    links take it off them.  With 1,500 links (and on level 1 with 120) the row
    exceeds the sparse product's scratch rows and the product is formed in
    two passes.  Tolerance: the row's sums have up to 1,500 terms of one sign,
    each rounded (1,500 x 2^-53 = 1.7e-13, and as much for the oracle's)."""
    import torch

    import paper_1810_08572_amd as ppe

    m = box_mesh(shape, jitter=0.1, seed=5)
    rng = np.random.default_rng(links)
    hub = m.n_cells // 2
    near = set(m.owner[m.neigh == hub]) | set(m.neigh[m.owner == hub]) | {hub}
    far = rng.permutation([c for c in range(m.n_cells) if c not in near])[:links]
    owner = np.concatenate([m.owner, np.full(links, hub)]).astype(np.int32)
    neigh = np.concatenate([m.neigh, far]).astype(np.int32)
    c0 = face_coeff(m, 2400.0)
    c = np.concatenate([c0, np.full(links, 1e-4 * c0[m.neigh >= 0].mean())])
    f = np.ones(m.n_cells)
    inner = neigh >= 0
    deg = np.bincount(np.concatenate([owner[inner], neigh[inner]]), minlength=m.n_cells)
    assert deg.max() == 4 + links
    sy = assembly.masked_system(m.n_cells, owner, neigh, c, f)
    H = amg.build_hierarchy(sy.A)
    assert len(H.levels) >= 2
    s = ppe.Solver()
    s.set_mesh(m.n_cells, to_dev(owner, torch.int32), to_dev(neigh, torch.int32))
    s.assemble(to_dev(c, torch.float64), to_dev(f, torch.float64))
    assert s.n_levels() == len(H.levels)
    for lvl, lev in enumerate(H.levels):
        n = lev.A.shape[0]
        A = csr(*s.level_matrix(lvl), (n, n))
        assert A.nnz == lev.A.nnz and rel_max(A, lev.A) <= 3.4e-13, lvl
        if lvl < len(H.levels) - 1:
            assert np.array_equal(s.aggregates(lvl).cpu().numpy(), lev.agg), lvl
            P = csr(*s.prolongator(lvl), lev.P.shape)
            if lvl == 0:
                assert (np.diff(P.indptr).max() > 256) == (links == 1500)
            assert rel_max(P, lev.P) <= 3.4e-13, lvl
    # and the solve on rows of these widths: the residual the oracle recomputes
    b = rng.normal(size=m.n_cells)
    b -= b.mean()
    res = s.solve(to_dev(b, torch.float64))
    assert res.status == 0
    assert assembly.relative_residual(sy, b, res.p.cpu().numpy()) <= 1e-10
    s.close()


def test_hierarchy_after_another_mesh_on_the_same_solver():
    """A chain of 200 cells, then a 40^3 cube, on one solver: the second
    setup reuses the first one's level buffers, MIS-2 batch counts and
    launch state, and must still give the oracle's hierarchy exactly."""
    import torch

    import paper_1810_08572_amd as ppe

    cm = 16
    s = ppe.Solver(coarse_max=cm)
    for m in (box_mesh((200, 1, 1), jitter=0.1, seed=1), box_mesh((40, 40, 40), jitter=0.1, seed=0)):
        f, c = np.ones(m.n_cells), face_coeff(m, 2400.0)
        sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
        H = amg.build_hierarchy(sy.A, coarse_max=cm)
        s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
        s.assemble(to_dev(c, torch.float64), to_dev(f, torch.float64))
        assert s.n_levels() == len(H.levels)
        for lvl, lev in enumerate(H.levels):
            n = lev.A.shape[0]
            A = csr(*s.level_matrix(lvl), (n, n))
            assert A.nnz == lev.A.nnz and rel_max(A, lev.A) <= 1e-13, lvl
            if lvl < len(H.levels) - 1:
                assert np.array_equal(s.aggregates(lvl).cpu().numpy(), lev.agg), lvl
        r = np.random.default_rng(8).normal(size=sy.n_active)
        z = s.apply_vcycle(to_dev(r, torch.float64)).cpu().numpy()
        assert np.linalg.norm(z - amg.vcycle(H, r)) <= 1e-12 * np.linalg.norm(z)
    s.close()


@pytest.mark.parametrize("cells", [8124, 8140, 8177, 8179, 8192])
def test_hierarchy_of_a_chain_that_fills_lds(cells):
    """MIS-2 of a small level in one workgroup takes 20 bytes of LDS per cell
    of a chain beside the kernel's own: the longest chain that does, and the
    lengths around the limit of 160 KB without and with the latter."""
    import torch

    import paper_1810_08572_amd as ppe

    m = box_mesh((cells, 1, 1), jitter=0.1, seed=2)
    f, c = np.ones(m.n_cells), face_coeff(m, 2400.0)
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    H = amg.build_hierarchy(sy.A)
    s = ppe.Solver()
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    s.assemble(to_dev(c, torch.float64), to_dev(f, torch.float64))
    assert s.n_levels() == len(H.levels)
    for lvl, lev in enumerate(H.levels[:-1]):
        assert np.array_equal(s.aggregates(lvl).cpu().numpy(), lev.agg), lvl
    s.close()


def test_products_whose_rows_outgrow_the_scratch():
    """A beam's second level has rows of 300 to 500 columns throughout: its
    R A P is formed in two passes at once, which the longest row of A P (four
    times as many columns pass the 256 of a scratch row) gives away."""
    import torch

    import paper_1810_08572_amd as ppe

    m = box_mesh((200, 20, 10), jitter=0.1, seed=1)
    f, c = np.ones(m.n_cells), face_coeff(m, 2400.0)
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    H = amg.build_hierarchy(sy.A, coarse_max=100)
    AP = (H.levels[1].A @ H.levels[1].P).tocsr()
    assert H.levels[2].A.shape[0] > 512 and 4 * np.diff(AP.indptr).max() > 256
    assert np.median(np.diff(H.levels[2].A.tocsr().indptr)) > 256
    s = ppe.Solver(coarse_max=100)
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    s.assemble(to_dev(c, torch.float64), to_dev(f, torch.float64))
    assert s.n_levels() == len(H.levels)
    for lvl, lev in enumerate(H.levels):
        A = csr(*s.level_matrix(lvl), lev.A.shape)
        # as test_hierarchy_matches_oracle: summation order only
        assert A.nnz == lev.A.nnz and rel_max(A, lev.A) <= 1e-13, lvl
    s.close()


@pytest.mark.parametrize("shape,shift,narrow", [((200, 20, 10), 0.0, True), ((200, 20, 10), 2.0, True),
                                                ((40, 40, 40), 0.0, False), ((20, 20, 20), 0.0, False)])
def test_transposes_on_both_sides_of_the_narrow_rule(shape, shift, narrow):
    """Prolongators of at most 1,024 columns and over 8 M columns times
    entries: transposed column by column up to 256 times the square of their
    mean column, by the general path beyond.  The transpose is the left factor
    of the next level's operator."""
    import scipy.sparse as sp
    import torch

    import paper_1810_08572_amd as ppe

    m = box_mesh(shape, jitter=0.1, seed=1)
    f, c = np.ones(m.n_cells), face_coeff(m, 2400.0)
    A = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f).A
    s = ppe.Solver(coarse_max=100)
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    if shift:
        d = np.full(m.n_cells, shift * np.median(c))
        k = m.neigh >= 0
        o, q, v = m.owner[k], m.neigh[k], c[k]
        A = sp.coo_matrix((np.concatenate([v, v, -v, -v, d]),
                           (np.concatenate([o, q, o, q, np.arange(m.n_cells)]),
                            np.concatenate([o, q, q, o, np.arange(m.n_cells)]))),
                          shape=(m.n_cells, m.n_cells)).tocsr()
        s.assemble_shifted(to_dev(c, torch.float64), to_dev(d, torch.float64))
    else:
        s.assemble(to_dev(c, torch.float64), to_dev(f, torch.float64))
    H = amg.build_hierarchy(A, coarse_max=100)
    sides = [P.shape[1] ** 3 <= 256 * P.nnz for P in (lev.P for lev in H.levels[:-1])
             if P.shape[1] <= 1024 and P.shape[1] * P.nnz > 8 << 20]
    assert sides == [narrow]
    assert s.n_levels() == len(H.levels)
    for lvl, lev in enumerate(H.levels):
        got = csr(*s.level_matrix(lvl), lev.A.shape)
        # as test_hierarchy_matches_oracle: summation order only
        assert got.nnz == lev.A.nnz and rel_max(got, lev.A) <= 1e-13, lvl
    s.close()
