"""Device memory from a caller's allocator that promises no more than it was
asked for: blocks cut to the byte from one arena, filled gaps between them.
Whatever the library runs, no gap is written.  And an allocator that has no
large block left: what the library can do without is not asked for twice."""
import ctypes

import numpy as np
import pytest

import paper_1810_08572_amd as ppe
from oracle import amg, assembly
from synth import al_alloy, box_mesh, face_coeff, fl_linear_x, rhs_uniform, t_wall_layer
from tests.gpu_util import csr, rel_max, to_dev, torch_dev

pytestmark = pytest.mark.gpu

FILL, GAP, ALIGN = 0xA5, 256, 256


class Arena:
    """Blocks of exactly the bytes asked for, never handed out twice."""

    def __init__(self, size):
        import torch

        self.mem = torch.full((size,), FILL, dtype=torch.uint8, device=torch_dev())
        self.base, self.size, self.at = self.mem.data_ptr(), size, 0
        self.blocks = []  # (offset, bytes)

        def _alloc(nbytes, stream, ctx):
            if self.at + nbytes + GAP > self.size:
                return None
            at = self.at
            self.blocks.append((at, int(nbytes)))
            self.at = (at + nbytes + GAP + ALIGN - 1) // ALIGN * ALIGN
            return self.base + at

        self._alloc = ppe.ALLOC_FN(_alloc)
        self._free = ppe.FREE_FN(lambda ptr, ctx: None)

    def install(self, o):
        o.alloc = ctypes.cast(self._alloc, ctypes.c_void_p)
        o.free = ctypes.cast(self._free, ctypes.c_void_p)
        o.alloc_ctx = None

    def check(self):
        """Every byte outside the blocks still holds the fill value."""
        import torch

        torch.cuda.synchronize()
        h = self.mem[:self.at + GAP].cpu().numpy()
        free = np.ones(h.size, dtype=bool)
        for at, n in self.blocks:
            free[at:at + n] = False
        bad = np.nonzero(free & (h != FILL))[0]
        if bad.size:
            before = [b for b in self.blocks if b[0] <= bad[0]][-1]
            raise AssertionError(f"{bad.size} bytes written outside their blocks, the first "
                                 f"{bad[0] - before[0]} bytes into a block of {before[1]}")
        assert len(self.blocks) > 20


def _f64(*arrays):
    import torch

    return [to_dev(a, torch.float64) for a in arrays]


# 44^3 cells: past the limits below which the component search and the scans
# take their short forms
@pytest.mark.parametrize("shape,opts", [
    ((10, 9, 8), {}), ((16, 14, 12), {"coarse_max": 8, "autotune": True}),
    ((20, 16, 18), {"precision": "mixed"}), ((24, 20, 22), {"smoother": "l1jacobi"}),
    ((24, 20, 22), {"coarse_reuse": 2}), ((44, 44, 44), {})])
def test_solver_writes_stay_in_their_blocks(shape, opts):
    import torch

    arena = Arena(1 << 29)
    m = box_mesh(shape, jitter=0.1, seed=1, mode="node")
    c = face_coeff(m, 2400.0)
    s = ppe.Solver(allocator=arena, **opts)
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    cd, = _f64(c)
    for x0 in (0.3, 0.35):
        fl = fl_linear_x(m.cell_centre, x0=x0)
        b, f = _f64(rhs_uniform(m.n_cells, seed=1, center_mask=fl > 0), fl)
        s.assemble(cd, f)
        for _ in range(5):  # with captured iterations
            p = s.solve(b).p
        s.solve(b, x0=p)
    arena.check()
    s.set_geometry(to_dev(m.nodes, torch.float64), to_dev(m.extra["face_nodes"], torch.int32),
                   to_dev(m.extra["cell_nodes"], torch.int32), *_f64(m.cell_centre, m.face_area))
    u = np.random.default_rng(2).normal(size=(m.n_cells, 3))
    s.project(cd, *_f64(u), 2400.0, 1e-3)
    shift, = _f64(np.full(m.n_cells, float(np.median(c))))
    s.assemble_shifted(cd, shift)
    s.solve(b)
    s.refresh_shift(cd, shift)
    s.solve(b)
    arena.check()


@pytest.mark.parametrize("shape", [(8, 7, 6), (20, 16, 18)])
def test_time_step_writes_stay_in_their_blocks(shape):
    import torch

    arena = Arena(1 << 29)
    m = box_mesh(shape, jitter=0.0, seed=1, lengths=tuple(0.01 * k / max(shape) for k in shape))
    fw = ppe.Flow(allocator=arena)
    fw.set_mesh(to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32), *_f64(m.nodes),
                to_dev(m.extra["face_nodes"], torch.int32),
                to_dev(m.extra["cell_nodes"], torch.int32),
                *_f64(m.cell_centre, m.face_area, m.face_centre, m.cell_volume))
    props = al_alloy(T_wall=600.0, T_ref=950.0)
    T, = _f64(t_wall_layer(m, 600.0, 950.0, 0.0008))
    fw.run(props, fw.new_state(T, props=props), 1e-3, 2)
    arena.check()


class Few(ppe.TorchAllocator):
    """PyTorch's allocator, but for blocks of more than `most` bytes."""

    def __init__(self, most):
        super().__init__(torch_dev())
        self.refused = 0
        take = self._alloc

        def _alloc(nbytes, stream, ctx):
            if nbytes > most:
                self.refused += 1
                return None
            return take(nbytes, stream, ctx)

        self._few = ppe.ALLOC_FN(_alloc)

    def install(self, o):
        super().install(o)
        o.alloc = ctypes.cast(self._few, ctypes.c_void_p)


# 22^3 cells: about 1,000 coarse rows, whose product's scratch rows take 1.0 MB
# of columns and 2.1 MB of values (one eighth more asked for); everything else
# the assembly asks for, the ELL copy and A P of 10,648 rows, is below 1 MB.
# One limit refuses the values alone, one both.
@pytest.mark.parametrize("most", [1 << 20, 3 << 19])
def test_products_without_memory_for_scratch_rows(most):
    import torch

    m = box_mesh((22, 22, 22), jitter=0.1, seed=0, mode="node")
    f, c = np.ones(m.n_cells), face_coeff(m, 2400.0)
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, f)
    H = amg.build_hierarchy(sy.A, coarse_max=100)
    few = Few(most)
    s = ppe.Solver(allocator=few, coarse_max=100)
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    for _ in range(2):
        s.assemble(*_f64(c, f))
        assert few.refused > 0
        assert s.n_levels() == len(H.levels)
        for lvl, lev in enumerate(H.levels):
            A = csr(*s.level_matrix(lvl), lev.A.shape)
            # as the hierarchy's parity tests: summation order only
            assert A.nnz == lev.A.nnz and rel_max(A, lev.A) <= 1e-13, lvl
    b = rhs_uniform(m.n_cells, seed=1, center_mask=f > 0)
    p = s.solve(*_f64(b)).p.cpu().numpy()
    assert assembly.relative_residual(sy, b, p) <= 1e-10
    s.close()


def test_workspace_of_the_dense_coarse_operator():
    """Level 1 of this shifted system (1,861 rows) gets its V-cycle as one
    matrix of 28 MB; forming it takes blocks of three vectors of that level and
    two of the next per column, 100 MB and an eighth of slack, and no more."""
    import torch

    m = box_mesh((27, 27, 27), jitter=0.05, seed=1)
    c = face_coeff(m, 2400.0)
    few = Few(120 << 20)
    s = ppe.Solver(allocator=few)
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    cd, shift, b = _f64(c, np.full(m.n_cells, 0.5 * float(np.median(c))),
                        np.random.default_rng(0).normal(size=m.n_cells))
    s.assemble_shifted(cd, shift)
    assert s.level_info(1)["n"] in range(1500, 2049)
    assert few.refused == 0
    assert s.solve(b).stats["rel_residual"] <= 1e-10
    s.close()
