"""A small coarse level's V-cycle formed as one dense matrix (of a pressure
system past the first coarse level, of a shifted system on any): the whole
V-cycle stays the oracle's to FP64 rounding, whatever the smoother, its degree,
the precision, the depth below the level and the mask."""
import copy

import numpy as np
import pytest

from oracle import amg, assembly
from synth import box_mesh, fl_linear_x
from tests.gpu_util import case, gpu_solver, to_dev

pytestmark = pytest.mark.gpu

# as the parity tests of the level-by-level V-cycle: summation order only
VCYCLE_RTOL = 1e-12


def _rounded(H):
    G = copy.deepcopy(H)
    q = lambda a: a.astype(np.float32).astype(np.float64)
    for lev in G.levels:
        lev.A, lev.diag = q(lev.A), q(lev.diag)
        if lev.P is not None:
            lev.P, lev.R = q(lev.P), q(lev.R)
    return G


def _check(s, H, n, seed):
    import torch

    r = np.random.default_rng(seed).normal(size=n)
    z = s.apply_vcycle(to_dev(r, torch.float64)).cpu().numpy()
    zr = amg.vcycle(H, r)
    assert np.linalg.norm(z - zr) <= VCYCLE_RTOL * np.linalg.norm(zr)


OPTS = [{}, {"coarse_max": 8}, {"coarse_max": 40, "cheb_degree": 1},
        {"cheb_degree": 3, "coarse_max": 8}, {"smoother": "l1jacobi", "coarse_max": 8},
        {"smoother": "l1jacobi", "cheb_degree": 1, "coarse_max": 8}, {"precision": "mixed"},
        {"precision": "mixed", "coarse_max": 8}, {"autotune": True, "coarse_max": 8}]


def _oracle(A, opts):
    H = amg.build_hierarchy(A, coarse_max=opts.get("coarse_max", 512),
                            degree=opts.get("cheb_degree", 2),
                            smoother=opts.get("smoother", "chebyshev"))
    return _rounded(H) if opts.get("precision") == "mixed" else H


# 24^3: levels of 9702, 958 and 46 rows (coarse_max 8 goes on below 46, and
# the third level's V-cycle is one matrix)
@pytest.mark.parametrize("opts", OPTS)
def test_pressure_vcycle(opts):
    import torch

    m, f, c, b = case(shape=(24, 24, 24), fl="front")
    s = gpu_solver(m, f, c, **opts)
    for fl in (f, fl_linear_x(m.cell_centre)):  # a new mask: nothing of the old matrices
        s.assemble(to_dev(c, torch.float64), to_dev(fl, torch.float64))
        sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, fl)
        _check(s, _oracle(sy.A, opts), sy.n_active, 1)
        for _ in range(3):  # captured iterations run the same operator
            p = s.solve(to_dev(b, torch.float64)).p.cpu().numpy()
            assert assembly.relative_residual(sy, b, p) <= 1e-10


# a shifted system takes the matrix on its first coarse level (12^3: about 500
# rows, 20 x 16 x 18: about 1500, an odd number of them)
@pytest.mark.parametrize("shape", [(12, 11, 13), (20, 16, 18)])
@pytest.mark.parametrize("opts", [{"coarse_max": 100}, {"coarse_max": 8, "precision": "mixed"},
                                  {"coarse_max": 100, "cheb_degree": 1}])
def test_shifted_vcycle(opts, shape):
    import scipy.sparse as sp
    import torch

    m = box_mesh(shape, jitter=0.1, seed=1)
    _, _, c, _ = case(mesh=m, fl="ones")
    inner = m.neigh >= 0
    o, q, v = m.owner[inner], m.neigh[inner], c[inner]
    n = m.n_cells
    L = sp.coo_matrix((np.concatenate([v, v, -v, -v]),
                       (np.concatenate([o, q, o, q]), np.concatenate([o, q, q, o]))),
                      shape=(n, n)).tocsr()
    rng = np.random.default_rng(3)
    d = np.median(v) * rng.uniform(0.5, 2.0, size=n)
    s = gpu_solver(m, np.ones(n), c, **opts)
    s.assemble_shifted(to_dev(c, torch.float64), to_dev(d, torch.float64))
    H = _oracle((L + sp.diags(d)).tocsr(), opts)
    _check(s, H, n, 5)
    # a refreshed diagonal changes the finest level only
    d2 = d * rng.uniform(0.8, 1.25, size=n)
    s.refresh_shift(to_dev(c, torch.float64), to_dev(d2, torch.float64))
    b = rng.normal(size=n)
    x = s.solve(to_dev(b, torch.float64)).p.cpu().numpy()
    r = b - (L + sp.diags(d2)) @ x
    assert np.linalg.norm(r) <= 1e-10 * np.linalg.norm(b)


def test_kept_coarse_levels_keep_the_dense_operator():
    import torch

    m = box_mesh((24, 24, 24), jitter=0.1, seed=0)
    f = fl_linear_x(m.cell_centre, x0=0.2)
    _, _, c, b = case(mesh=m, fl=f)
    bd, cd = to_dev(b, torch.float64), to_dev(c, torch.float64)
    moved = to_dev(fl_linear_x(m.cell_centre, x0=0.23), torch.float64)
    s = gpu_solver(m, f, c, coarse_reuse=4, coarse_max=8)
    s.solve(bd)
    s.assemble(cd, moved)
    assert s.stats()["coarse_reused"] == 1
    sy0 = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, moved.cpu().numpy())
    row = np.full(m.n_cells, -1)
    row[sy0.perm] = np.arange(sy0.n_active)
    pinned = np.zeros(sy.n_active, dtype=bool)
    pinned[sy.pinned] = True
    H = amg.reuse_coarse_levels(_oracle(sy0.A, {"coarse_max": 8}), sy.A, row[sy.perm], pinned)
    _check(s, H, sy.n_active, 4)
