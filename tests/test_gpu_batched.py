"""Batched uncertainty samples: meshes of uneven size solved in one call as
a block-diagonal union, each sample with its own CG scalars and stopping
test.  Every sample meets the single-solve bars (residual <= 1e-10, L2
error <= 1e-9 against its own exact solve); changing one sample's
right-hand side leaves every other sample's pressure bitwise unchanged."""
import numpy as np
import pytest

from oracle import assembly, direct
from synth import batch_samples, box_mesh, concat_meshes, face_coeff, rhs_uniform, uq_front_fl
from tests.gpu_util import to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _batch(n=6, t=0.12, seed=11):
    samples = batch_samples(n, seed=seed, side_range=(6, 14))
    meshes = [box_mesh((sm["side"],) * 3, jitter=0.1, seed=k) for k, sm in enumerate(samples)]
    fls = [uq_front_fl(m.cell_centre, sm, t, 0.2) for m, sm in zip(meshes, samples)]
    u = concat_meshes(meshes)
    fl = np.concatenate(fls)
    c = face_coeff(u, 2400.0)
    bs = [rhs_uniform(m.n_cells, seed=100 + k, center_mask=f > 0) for k, (m, f) in
          enumerate(zip(meshes, fls))]
    return meshes, fls, u, fl, c, bs


def _solver(u, fl, c, **kw):
    import torch

    import paper_1810_08572_amd as ppe

    torch_dev()
    s = ppe.Solver(**kw)
    s.set_mesh(u.n_cells, to_dev(u.owner, torch.int32), to_dev(u.neigh, torch.int32))
    s.set_segments(u.extra["cell_offsets"])
    s.assemble(to_dev(c, torch.float64), to_dev(fl, torch.float64))
    return s


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_each_sample_meets_single_solve_bars(precision):
    import torch

    meshes, fls, u, fl, c, bs = _batch()
    s = _solver(u, fl, c, precision=precision)
    res = s.solve(to_dev(np.concatenate(bs), torch.float64))
    p = res.p.cpu().numpy()
    its, rrs = s.segment_stats()
    off = u.extra["cell_offsets"]
    for k, m in enumerate(meshes):
        ck = face_coeff(m, 2400.0)
        sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, ck, fls[k])
        pk = p[off[k]:off[k + 1]]
        ref = direct.solve_sparse(sy, bs[k])
        assert assembly.relative_residual(sy, bs[k], pk) <= 1e-10, k
        assert np.linalg.norm(pk - ref) <= 1e-9 * max(np.linalg.norm(ref), 1e-300), k
        assert rrs[k] <= 1e-10 and its[k] >= 1
    assert res.stats["iterations"] == max(its)


def test_rhs_perturbation_is_isolated():
    import torch

    meshes, fls, u, fl, c, bs = _batch()
    s = _solver(u, fl, c)
    p1 = s.solve(to_dev(np.concatenate(bs), torch.float64)).p.cpu().numpy()
    its1, _ = s.segment_stats()
    bs2 = list(bs)
    bs2[2] = bs[2] * -3.0 + 0.1 * rhs_uniform(len(bs[2]), seed=999)
    p2 = s.solve(to_dev(np.concatenate(bs2), torch.float64)).p.cpu().numpy()
    its2, _ = s.segment_stats()
    off = u.extra["cell_offsets"]
    for k in range(len(meshes)):
        a, b = p1[off[k]:off[k + 1]], p2[off[k]:off[k + 1]]
        if k == 2:
            assert not np.array_equal(a, b)
        else:
            assert np.array_equal(a, b), k
            assert its1[k] == its2[k]


def test_zero_rhs_sample_and_bad_segments():
    import torch

    import paper_1810_08572_amd as ppe

    meshes, fls, u, fl, c, bs = _batch(n=3)
    s = _solver(u, fl, c)
    bs[1] = np.zeros_like(bs[1])
    res = s.solve(to_dev(np.concatenate(bs), torch.float64))
    off = u.extra["cell_offsets"]
    assert not res.p.cpu().numpy()[off[1]:off[2]].any()
    its, _ = s.segment_stats()
    assert its[1] == 0 and its[0] > 0
    bad = list(off)
    bad[1] += 5   # cuts through sample 0: faces join two samples
    with pytest.raises(ppe.PpeError) as e:
        s.set_segments(bad)
    assert e.value.status == ppe.PPE_ERR_ARG


# 27 and 64 rows of a 512-thread tile: the passes of an iteration run one by one
# (below 100 rows per tile); 216 rows: the residual's update takes the first
# smoothing steps along
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sides", [[3] * 180, [4] * 60, [3, 4] * 70, [6] * 30])
def test_many_samples_of_a_few_cells(sides, precision):
    import torch

    meshes = [box_mesh((k,) * 3, jitter=0.1, seed=q) for q, k in enumerate(sides)]
    u = concat_meshes(meshes)
    c, fl = face_coeff(u, 2400.0), np.ones(u.n_cells)
    b = np.concatenate([rhs_uniform(m.n_cells, seed=q, center_mask=np.ones(m.n_cells, bool))
                        for q, m in enumerate(meshes)])
    s = _solver(u, fl, c, precision=precision)
    assert s.n_levels() >= 2
    off = u.extra["cell_offsets"]
    for _ in range(5):  # with captured iterations
        p = s.solve(to_dev(b, torch.float64)).p.cpu().numpy()
    for q, m in enumerate(meshes):
        sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, face_coeff(m, 2400.0),
                                    np.ones(m.n_cells))
        bq, pq = b[off[q]:off[q + 1]], p[off[q]:off[q + 1]]
        assert assembly.relative_residual(sy, bq, pq) <= 1e-10, q
        ref = direct.solve_dense(sy, bq)
        assert np.linalg.norm(pq - ref) <= 1e-9 * np.linalg.norm(ref), q
