"""GPU parity of the collocation wrapper (section 3, Eq. 27-28) against the
oracle:

- least-squares coefficients, evaluation at Latin-hypercube points and the
  mean / variance / Sobol indices of many outputs at once, against numpy's
  least squares and the oracle's statistics (1e-12), with term counts,
  sample counts and output counts that cross the kernel's tiles;
- a collocation over batched pressure solves: the fields of 27 tensor
  samples of three inputs (melt and wall temperature normal, liquidus shift
  uniform) on one mesh, fitted on the GPU and by the oracle from the same
  solved fields;
- too few or repeated points are rejected.
"""
import numpy as np
import pytest

from oracle import uq
from synth import box_mesh, concat_meshes, face_coeff, latin_hypercube, rhs_smooth_series, uq_front_fl
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu
KINDS = ["normal", "normal", "uniform"]
OK = [uq.NORMAL, uq.NORMAL, uq.UNIFORM]


def test_fit_eval_stats_match_oracle():
    import torch

    import paper_1810_08572_amd as ppe

    q = ppe.PolynomialChaos(KINDS, 3)
    assert q.n_terms == 20
    X, _ = q.nodes("smolyak", 4)
    assert X.shape[0] == 69
    rng = np.random.default_rng(2)
    n_out = 5003
    Y = rng.normal(size=(X.shape[0], n_out))
    W = q.fit(X, to_dev(Y, torch.float64)).cpu().numpy()
    al = uq.total_degree_indices(3, 3)
    Wo = uq.fit(uq.vandermonde(OK, al, X), Y)
    assert np.abs(W - Wo).max() <= 1e-12 * np.abs(Wo).max()
    T, _ = latin_hypercube(KINDS, 60, seed=4)
    Ye = q.eval(T, to_dev(Wo, torch.float64)).cpu().numpy()
    Yo = uq.vandermonde(OK, al, T) @ Wo
    assert np.abs(Ye - Yo).max() <= 1e-12 * np.abs(Yo).max()
    mean, var, first, total = [t.cpu().numpy() for t in q.stats(to_dev(Wo, torch.float64))]
    mo, vo, fo, to = uq.statistics(al, Wo)
    assert np.abs(mean - mo).max() <= 1e-14 * np.abs(mo).max()
    assert np.abs(var - vo).max() <= 1e-12 * np.abs(vo).max()
    assert np.abs(first - fo).max() <= 1e-12 and np.abs(total - to).max() <= 1e-12


def test_collocation_of_batched_pressure_solves():
    import torch

    import paper_1810_08572_amd as ppe

    q = ppe.PolynomialChaos(KINDS, 2)
    X, _ = q.nodes("tensor", 3)  # 27 samples, as in the paper's three-input table
    m = box_mesh((16, 16, 16), lengths=(0.01,) * 3, jitter=0.1, seed=0)
    u = concat_meshes([m] * X.shape[0])
    fls, bs = [], []
    for x in X:
        sm = dict(t_melt=950.0 + 10.0 * x[0], t_wall=600.0 + 20.0 * x[1], d_liq=5.0 * x[2])
        f = uq_front_fl(m.cell_centre, sm, 0.03, 0.05, length=0.01)
        fls.append(f)
        bs.append(rhs_smooth_series(m.cell_centre, 0.03, seed=5, center_mask=f > 0))
    s = ppe.Solver()
    s.set_mesh(u.n_cells, to_dev(u.owner, torch.int32), to_dev(u.neigh, torch.int32))
    s.set_segments(u.extra["cell_offsets"])
    s.assemble(to_dev(face_coeff(u, 2400.0), torch.float64), to_dev(np.concatenate(fls), torch.float64))
    res = s.solve(to_dev(np.concatenate(bs), torch.float64))
    its, rr = s.segment_stats()
    assert max(rr) <= 1e-10
    Y = res.p.reshape(X.shape[0], m.n_cells)
    W = q.fit(X, Y).cpu().numpy()
    al = uq.total_degree_indices(3, 2)
    Wo = uq.fit(uq.vandermonde(OK, al, X), Y.cpu().numpy())
    assert np.abs(W - Wo).max() <= 1e-12 * np.abs(Wo).max()
    mean, var, first, total = [t.cpu().numpy() for t in q.stats(to_dev(Wo, torch.float64))]
    # the front depth depends on the wall and melt temperatures: the cells
    # whose pressure varies at all are sensitive to them
    varying = var > 1e-6 * var.max()
    assert varying.sum() > 100
    f, t = first[:, varying], total[:, varying]
    assert np.all(f >= 0) and np.all(f <= t + 1e-12) and np.all(t <= 1 + 1e-12)
    assert np.all(f.sum(axis=0) <= 1 + 1e-12)
    print(f"27 samples x {m.n_cells} cells: mean PCG iterations {np.mean(its):.1f}, "
          f"cells with varying pressure {varying.sum()}", flush=True)


def test_rejects_too_few_or_repeated_points():
    import torch

    import paper_1810_08572_amd as ppe

    q = ppe.PolynomialChaos(KINDS, 2)  # 10 terms
    Y = to_dev(np.ones((8, 4)), torch.float64)
    with pytest.raises(ppe.PpeError) as e:
        q.fit(np.zeros((8, 3)), Y)
    assert e.value.status == ppe.PPE_ERR_ARG
    X = np.repeat(np.random.default_rng(0).normal(size=(4, 3)), 3, axis=0)  # 12 points, 4 distinct
    with pytest.raises(ppe.PpeError) as e:
        q.fit(X, to_dev(np.ones((12, 4)), torch.float64))
    assert e.value.status == ppe.PPE_ERR_ARG


def test_smallest_expansions():
    """Degree 0 (the mean only) from one node; one input; the smallest
    Smolyak grid; a single output column."""
    import torch

    import paper_1810_08572_amd as ppe

    q = ppe.PolynomialChaos(["normal"], 0)
    X, w = q.nodes("smolyak", 1)
    assert X.shape == (1, 1) and X[0, 0] == 0.0 and w[0] == 1.0
    Y = to_dev(np.array([[3.5, -1.0]]), torch.float64)
    W = q.fit(X, Y).cpu().numpy()
    assert np.array_equal(W, np.array([[3.5, -1.0]]))
    mean, var, first, total = [t.cpu().numpy() for t in q.stats(to_dev(W, torch.float64))]
    assert np.array_equal(mean, [3.5, -1.0]) and np.all(var == 0) and np.all(total == 0)
    q = ppe.PolynomialChaos(["uniform"], 4)
    X, _ = q.nodes("tensor", 5)
    x = X[:, 0]
    y = 1.0 + 2.0 * x - 0.5 * x ** 4  # in the span of the basis
    W = q.fit(X, to_dev(y[:, None], torch.float64))
    T = np.linspace(-1, 1, 7)[:, None]
    Ye = q.eval(T, W).cpu().numpy()[:, 0]
    assert np.abs(Ye - (1.0 + 2.0 * T[:, 0] - 0.5 * T[:, 0] ** 4)).max() <= 1e-13


# the matrix-core product's edges (16-row and 16-column tiles, 64 rows and 64
# columns of a workgroup, 32 staged columns), the reflections of one column,
# of more columns than a workgroup's waves take at a time, and of a set whose
# factorisation does not fit in LDS (M K words and more)
@pytest.mark.parametrize("kinds,degree,M,n_out", [
    (["uniform"], 0, 1, 1), (["normal"], 1, 2, 17), (["uniform"] * 2, 3, 10, 64),
    (["uniform"] * 3, 4, 35, 65), (["normal", "uniform"], 5, 63, 15), (["uniform"] * 3, 5, 65, 130),
    (["uniform"] * 4, 4, 200, 33), (["uniform"] * 4, 5, 400, 70), (["uniform"] * 6, 3, 260, 5)])
def test_fit_eval_stats_at_tile_edges(kinds, degree, M, n_out):
    import torch

    import paper_1810_08572_amd as ppe

    ok = [uq.NORMAL if k == "normal" else uq.UNIFORM for k in kinds]
    q = ppe.PolynomialChaos(kinds, degree)
    X, _ = latin_hypercube(kinds, M, seed=M)
    Y = np.random.default_rng(M).normal(size=(M, n_out))
    al = uq.total_degree_indices(len(kinds), degree)
    V = uq.vandermonde(ok, al, X)
    # a backward-stable least-squares solution differs by eps times the
    # condition number (1 + its square times the residual): the bar of the
    # well-conditioned cases, 1e-12, scaled by it
    cond = np.linalg.cond(V)
    W = q.fit(X, to_dev(Y, torch.float64)).cpu().numpy()
    Wo = uq.fit(V, Y)
    assert np.abs(W - Wo).max() <= 1e-14 * (100 + cond ** 2) * np.abs(Wo).max()
    Ye = q.eval(X, to_dev(Wo, torch.float64)).cpu().numpy()
    assert np.abs(Ye - V @ Wo).max() <= 1e-13 * (np.abs(V) @ np.abs(Wo)).max()
    mean, var, first, total = [t.cpu().numpy() for t in q.stats(to_dev(Wo, torch.float64))]
    mo, vo, fo, to = uq.statistics(al, Wo)
    assert np.array_equal(mean, mo) and np.abs(var - vo).max() <= 1e-12 * np.abs(vo).max()
    assert np.abs(first - fo).max(initial=0) <= 1e-12 and np.abs(total - to).max(initial=0) <= 1e-12


def test_rank_deficient_fit_leaves_the_coefficients_alone():
    import torch

    import paper_1810_08572_amd as ppe

    q = ppe.PolynomialChaos(KINDS, 2)
    X = np.repeat(np.random.default_rng(0).normal(size=(4, 3)), 3, axis=0)
    Y = to_dev(np.ones((12, 70)), torch.float64)
    keep = torch.empty
    W = to_dev(np.full((q.n_terms, 70), 7.0), torch.float64)
    torch.empty = lambda *a, **k: W
    try:
        with pytest.raises(ppe.PpeError):
            q.fit(X, Y)
    finally:
        torch.empty = keep
    assert bool((W == 7.0).all())
    good = q.fit(q.nodes("tensor", 3)[0], to_dev(np.ones((27, 70)), torch.float64))
    assert abs(float(good[0, 0]) - 1.0) <= 1e-13


def test_more_outputs_than_one_launch_holds():
    """2^30 outputs and a few: more than one grid of the products and of the
    statistics takes (2^32 threads), so they go in parts of 2^29.  One constant
    term, so every result is its sample."""
    import torch

    import paper_1810_08572_amd as ppe

    n = (1 << 30) + 5
    q = ppe.PolynomialChaos(["uniform"], 0)
    X = np.zeros((1, 1))
    Y = torch.empty(1, n, dtype=torch.float64, device="cuda")
    Y[0] = torch.arange(n, device="cuda", dtype=torch.int32)
    W = q.fit(X, Y)
    assert torch.equal(W, Y)
    del Y
    mean, var, first, total = q.stats(W)
    assert torch.equal(mean, W[0])
    assert not bool(var.any() or first.any() or total.any())
    del mean, var, first, total
    assert torch.equal(q.eval(X, W), W)
    q.close()
    del W
    torch.cuda.empty_cache()


# the factorisation runs on the host below 4,000 + 40 K values (points x terms):
# both sides of that line, one term, as many points as terms
@pytest.mark.parametrize("kinds,degree,M", [
    (["uniform"], 0, 1), (["uniform"] * 2, 3, 10), (["uniform"] * 3, 3, 239),
    (["uniform"] * 3, 3, 240), (["uniform"] * 3, 5, 111), (["uniform"] * 3, 5, 112),
    (["uniform"] * 2, 9, 56), (["uniform"], 19, 241)])
def test_fit_on_host_and_device(kinds, degree, M):
    import torch

    import paper_1810_08572_amd as ppe

    q = ppe.PolynomialChaos(kinds, degree)
    X, _ = latin_hypercube(kinds, M, seed=M)
    Y = np.random.default_rng(M).normal(size=(M, 65))
    V = uq.vandermonde([uq.UNIFORM] * len(kinds), uq.total_degree_indices(len(kinds), degree), X)
    cond = np.linalg.cond(V)
    W = q.fit(X, to_dev(Y, torch.float64)).cpu().numpy()
    Wo = uq.fit(V, Y)
    # as test_fit_eval_stats_at_tile_edges
    assert np.abs(W - Wo).max() <= 1e-14 * (100 + cond ** 2) * np.abs(Wo).max()


# twelve points: factorised on the host; 250: on the device; 300: from global memory
@pytest.mark.parametrize("degree,M", [(2, 12), (5, 250), (5, 300)])
def test_a_refused_fit_writes_no_coefficient(degree, M):
    """Through the C entry point: points that repeat are refused as rank
    deficient, the coefficients stay, and the next fit is whole."""
    import ctypes

    import torch

    import paper_1810_08572_amd as ppe

    q = ppe.PolynomialChaos(KINDS, degree)
    lib, K, n = ppe.load_library(), q.n_terms, 70
    few = np.random.default_rng(0).normal(size=((K + 1) // 2, 3))
    X = np.ascontiguousarray(np.resize(few, (M, 3)))
    Y = to_dev(np.ones((M, n)), torch.float64)
    W = to_dev(np.full((K, n), 7.0), torch.float64)

    def fit(pts):
        return lib.ppe_pce_fit(q._h, len(pts), pts.ctypes.data_as(ctypes.c_void_p), n,
                               ctypes.c_void_p(Y.data_ptr()), ctypes.c_void_p(W.data_ptr()))

    assert fit(X) == ppe.PPE_ERR_ARG
    torch.cuda.synchronize()
    assert bool((W == 7.0).all())
    good = np.ascontiguousarray(latin_hypercube(KINDS, M, seed=1)[0])
    assert fit(good) == 0
    # a constant field: coefficient 1 of the constant term, 0 elsewhere
    assert float((W[0] - 1.0).abs().max()) <= 1e-10 and float(W[1:].abs().max()) <= 1e-10
