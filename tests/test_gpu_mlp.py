"""Learned warm start: the GPU network's FP32 loss and gradients match the
FP64 oracle; BF16 matrix-core inference matches the FP32 forward pass to
BF16 rounding; one Adam step matches the oracle's; the features match the
oracle's definition; and a network trained on snapshots the solver itself
produced reduces the iterations of held-out solves (the solve always ends at
the FP64 tolerance, whatever the initial guess)."""
import numpy as np
import pytest

from oracle import assembly, mlp as omlp
from synth import box_mesh, face_coeff, fl_growing_front, rhs_smooth_series
from tests.gpu_util import to_dev, torch_dev

pytestmark = pytest.mark.gpu

# FP32 forward/backward against FP64: the gradient of a mean over n rows of
# products of FP32-rounded layers agrees to ~sqrt(n) * 6e-8 * depth relative
BWD_RTOL = 1e-4
# BF16 activations/weights (8-bit mantissa, 2^-9 = 2e-3 relative rounding)
# through three rounded layers: a CPU emulation of exactly that rounding on
# the oracle's forward pass gives 3.0e-3 relative L2 for this network
BF16_RTOL = 1e-2
# the GPU's BF16 pass against that emulation: only FP32 summation order and
# the rare BF16 tie it moves differ
BF16_EMUL_RTOL = 1e-3


def _net(seed=0, width=128, hidden=3):
    import paper_1810_08572_amd as ppe
    import torch

    torch_dev()
    shapes = omlp.layer_shapes(10, width, hidden)
    theta = omlp.init_params(shapes, seed=seed)
    net = ppe.WarmStartNet(10, width, hidden)
    net.set_params(to_dev(theta.astype(np.float32), torch.float32))
    return net, shapes, theta.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("n", [1, 77, 5000])
def test_fp32_loss_and_gradient_match_oracle(n):
    import torch

    net, shapes, theta = _net()
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, 10)).astype(np.float32)
    T = rng.normal(size=n).astype(np.float32)
    loss, g = net.loss_grad(to_dev(X, torch.float32), to_dev(T, torch.float32))
    l_ref, g_ref = omlp.loss_and_grad(theta, shapes, X.astype(np.float64), T.astype(np.float64))
    assert abs(loss - l_ref) <= BWD_RTOL * l_ref
    g = g.cpu().numpy()
    assert np.linalg.norm(g - g_ref) <= BWD_RTOL * np.linalg.norm(g_ref)
    y = net.forward(to_dev(X, torch.float32)).cpu().numpy()
    y_ref, _, _ = omlp.forward(theta, shapes, X.astype(np.float64))
    assert np.abs(y - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max())


# edges of the 32 x 32 product tiles, of the 128-column workgroup tiles, of the
# staged depth (64) and of the gradient's row chunks (128 rows, 64 chunks)
@pytest.mark.parametrize("n,width,hidden", [(1, 1, 1), (31, 32, 2), (33, 33, 3), (129, 65, 1),
                                            (127, 128, 2), (8193, 100, 3), (500, 129, 2),
                                            (64, 300, 2), (40, 5, 18)])
def test_fp32_gradient_at_tile_edges(n, width, hidden):
    import torch

    net, shapes, theta = _net(seed=1, width=width, hidden=hidden)
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, 10)).astype(np.float32)
    T = rng.normal(size=n).astype(np.float32)
    loss, g = net.loss_grad(to_dev(X, torch.float32), to_dev(T, torch.float32))
    l_ref, g_ref = omlp.loss_and_grad(theta, shapes, X.astype(np.float64), T.astype(np.float64))
    assert abs(loss - l_ref) <= BWD_RTOL * l_ref
    at = 0
    for a, b in shapes:  # every layer's weights and biases by themselves
        for size in (a * b, a):
            ref = g_ref[at:at + size]
            got = g[at:at + size].cpu().numpy()
            assert np.linalg.norm(got - ref) <= BWD_RTOL * np.linalg.norm(ref) + 1e-7 * np.linalg.norm(g_ref)
            at += size
    assert at == net.n_params
    y = net.forward(to_dev(X, torch.float32)).cpu().numpy()
    y_ref, _, _ = omlp.forward(theta, shapes, X.astype(np.float64))
    assert np.abs(y - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max())


# narrow layers take tiles of 64 and 128 rows from 16,384 and 32,768 rows on:
# both sides of those lines and of the widths, ragged last tiles.  As above;
# the oracle's sums over the rows are in FP64, ours in FP32 chunks of rows
@pytest.mark.parametrize("n,width", [(16383, 64), (16385, 33), (16500, 64), (32767, 32),
                                     (32769, 1), (33000, 32), (40001, 17), (32768, 65)])
def test_fp32_narrow_layers(n, width):
    import torch

    net, shapes, theta = _net(seed=2, width=width, hidden=2)
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, 10)).astype(np.float32)
    T = rng.normal(size=n).astype(np.float32)
    Xd, Td = to_dev(X, torch.float32), to_dev(T, torch.float32)
    y_ref, _, _ = omlp.forward(theta, shapes, X.astype(np.float64))
    y = net.forward(Xd).cpu().numpy()
    assert np.abs(y - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max())
    loss, g = net.loss_grad(Xd, Td)
    l_ref, g_ref = omlp.loss_and_grad(theta, shapes, X.astype(np.float64), T.astype(np.float64))
    assert abs(loss - l_ref) <= BWD_RTOL * l_ref
    assert np.linalg.norm(g.cpu().numpy() - g_ref) <= BWD_RTOL * np.linalg.norm(g_ref)


def test_fp32_more_rows_than_one_launch_holds():
    """2^28 rows and a few: a layer's tiles are more than one grid takes (2^32
    threads), so its rows go in parts of 2^27; checked at both ends and around
    the parts' edges."""
    import torch

    import paper_1810_08572_amd as ppe

    n = (1 << 28) + 7
    shapes = omlp.layer_shapes(1, 33, 1)
    theta = omlp.init_params(shapes, seed=8).astype(np.float32)
    net = ppe.WarmStartNet(1, 33, 1)
    net.set_params(to_dev(theta, torch.float32))
    theta = theta.astype(np.float64)
    X = torch.rand(n, 1, device=torch_dev(), generator=torch.Generator(torch_dev()).manual_seed(8))
    y = net.forward(X)
    for a in (0, (1 << 27) - 500, (1 << 28) - 500, n - 1000):
        ref, _, _ = omlp.forward(theta, shapes, X[a:a + 1000].cpu().numpy().astype(np.float64))
        err = np.abs(y[a:a + 1000].cpu().numpy() - ref).max()
        assert err <= 1e-5 * max(1.0, np.abs(ref).max()), a
    net.close()
    del X, y
    torch.cuda.empty_cache()


# 100003 cells: more 32-cell tiles than one launch's waves, so waves stride
# over several tiles, with a ragged last tile
@pytest.mark.parametrize("n", [1, 32, 1000, 12345, 100003])
def test_bf16_inference_matches_fp32(n):
    import torch

    net, shapes, theta = _net(seed=3)
    X = to_dev(np.random.default_rng(1).normal(size=(n, 10)).astype(np.float32), torch.float32)
    y32 = net.forward(X).cpu().numpy()
    y16 = net.forward(X, bf16=True).cpu().numpy()
    assert np.linalg.norm(y16 - y32) <= BF16_RTOL * np.linalg.norm(y32)
    if n > 1:
        assert not np.array_equal(y16, y32)   # the BF16 path really ran
    ye = _bf16_forward(theta, shapes, X.cpu().numpy().astype(np.float64))
    assert np.linalg.norm(y16 - ye) <= BF16_EMUL_RTOL * np.linalg.norm(ye)


# the twelve waves of a workgroup, ragged tiles, and the depths whose weights
# fit in LDS (two to five hidden layers) or do not (six)
@pytest.mark.parametrize("hidden", [2, 4, 5, 6])
@pytest.mark.parametrize("n", [1, 31, 385, 13000])
def test_bf16_inference_depths(n, hidden):
    import torch

    net, shapes, theta = _net(seed=4, hidden=hidden)
    X = to_dev(np.random.default_rng(n).normal(size=(n, 10)).astype(np.float32), torch.float32)
    y = net.forward(X, bf16=True).cpu().numpy()
    ye = _bf16_forward(theta, shapes, X.cpu().numpy().astype(np.float64))
    assert np.linalg.norm(y - ye) <= BF16_EMUL_RTOL * np.linalg.norm(ye)


def test_bf16_inference_is_the_same_for_any_number_of_waves():
    """A workgroup runs eight or twelve waves, whichever needs fewer rounds:
    a cell's output does not depend on it, at and around the sizes where the
    choice turns (32 cells x 256 compute units x 8 or 12 waves)."""
    import torch

    net, shapes, theta = _net(seed=6)
    X = to_dev(np.random.default_rng(6).normal(size=(200000, 10)).astype(np.float32), torch.float32)
    y = net.forward(X, bf16=True)
    ye = _bf16_forward(theta, shapes, X[-3000:].cpu().numpy().astype(np.float64))
    assert np.linalg.norm(y[-3000:].cpu().numpy() - ye) <= BF16_EMUL_RTOL * np.linalg.norm(ye)
    for n in (257, 65536, 65537, 98304, 98305, 131073, 196609):
        assert torch.equal(net.forward(X[:n].contiguous(), bf16=True), y[:n]), n


def _bf16(a):
    """Round to the nearest BF16 (ties to even), returned as float64."""
    u = np.asarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


def _bf16_forward(theta, shapes, X):
    """The oracle's forward pass with the BF16 inference's roundings: every
    hidden activation and the width x width weights rounded to BF16, sums
    exact."""
    layers = omlp.unpack(theta, shapes)
    h = _bf16(omlp.silu(X @ layers[0][0].T + layers[0][1]))
    for W, b in layers[1:-1]:
        h = _bf16(omlp.silu(h @ _bf16(W).T + b))
    W, b = layers[-1]
    return (h @ W.T + b)[:, 0]


def test_adam_step_matches_oracle():
    import torch

    net, shapes, theta = _net(seed=5, width=32, hidden=2)
    rng = np.random.default_rng(0)
    X = rng.normal(size=(500, 10)).astype(np.float32)
    T = np.tanh(X[:, 0]).astype(np.float32)
    lr = 1e-3
    net.train_step(to_dev(X, torch.float32), to_dev(T, torch.float32), lr)
    new = net.get_params().cpu().numpy()
    _, g = omlp.loss_and_grad(theta, shapes, X.astype(np.float64), T.astype(np.float64))
    ref, _, _ = omlp.adam_step(theta, g, np.zeros_like(g), np.zeros_like(g), 1, lr)
    big = np.abs(g) > 1e-3 * np.abs(g).max()   # first Adam step ~ lr*sign(g): skip g ~ 0
    assert np.abs(new - ref)[big].max() <= 1e-2 * lr


def _series(m, c, steps, t0, seed, solver):
    """Run the solver through a smooth series; yields per-step tensors."""
    import torch

    dev = torch.device("cuda", 0)
    p_prev = torch.zeros(m.n_cells, dtype=torch.float64, device=dev)
    dp_prev = torch.zeros_like(p_prev)
    for k in range(steps):
        t = t0 + 1e-3 * k
        fl = fl_growing_front(m.cell_centre, t, 0.2, s_max=0.5)
        b = rhs_smooth_series(m.cell_centre, t, seed=seed, center_mask=fl > 0)
        yield k, fl, b, p_prev, dp_prev
        solver.assemble(to_dev(c, torch.float64), to_dev(fl, torch.float64))
        p = solver.solve(to_dev(b, torch.float64)).p.clone()
        dp_prev = p - p_prev
        p_prev = p


def test_features_match_oracle_definition():
    import torch

    import paper_1810_08572_amd as ppe

    torch_dev()
    m = box_mesh((11, 9, 7), jitter=0.1, seed=2)
    c = face_coeff(m, 2400.0)
    s = ppe.Solver()
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    fl = fl_growing_front(m.cell_centre, 0.05, 0.2)
    s.assemble(to_dev(c, torch.float64), to_dev(fl, torch.float64))
    rng = np.random.default_rng(4)
    dp, b = rng.normal(size=m.n_cells), rng.normal(size=m.n_cells)
    mu = np.zeros(10, np.float32)
    sg = np.ones(10, np.float32)
    F, scale = ppe.warm_start_features(s, to_dev(dp, torch.float64), to_dev(b, torch.float64),
                                       to_dev(c, torch.float64), to_dev(fl, torch.float64),
                                       to_dev(m.cell_volume, torch.float64),
                                       to_dev(mu, torch.float32), to_dev(sg, torch.float32))
    sy = assembly.masked_system(m.n_cells, m.owner, m.neigh, c, fl)
    pin_of = np.zeros(m.n_cells, dtype=np.int64)
    pin_of[sy.perm] = sy.comp
    Fr, sr = omlp.warm_start_features(m.n_cells, m.owner, m.neigh, c, fl, m.cell_volume, dp, b,
                                      pin_of)
    assert abs(scale - sr) <= 1e-14 * sr
    assert np.abs(F.cpu().numpy() - Fr).max() <= 1e-6


def test_features_of_cells_with_many_neighbours():
    """More than six neighbours (extra faces to in-plane diagonal cells): the
    plain neighbour loop, against the oracle's definition."""
    import torch

    import paper_1810_08572_amd as ppe

    torch_dev()
    m = box_mesh((9, 8, 7), jitter=0.1, seed=3)
    c0 = face_coeff(m, 2400.0)
    g = m.grid_index
    cell = {tuple(v): k for k, v in enumerate(g)}
    pairs = [(k, cell[(i + 1, j + 1, l)]) for k, (i, j, l) in enumerate(g)
             if (i + 1, j + 1, l) in cell]
    owner = np.concatenate([m.owner, [p[0] for p in pairs]]).astype(np.int32)
    neigh = np.concatenate([m.neigh, [p[1] for p in pairs]]).astype(np.int32)
    rng = np.random.default_rng(6)
    c = np.concatenate([c0, np.median(c0[m.neigh >= 0]) * rng.uniform(0.1, 0.5, size=len(pairs))])
    s = ppe.Solver()
    s.set_mesh(m.n_cells, to_dev(owner, torch.int32), to_dev(neigh, torch.int32))
    fl = fl_growing_front(m.cell_centre, 0.05, 0.2)
    s.assemble(to_dev(c, torch.float64), to_dev(fl, torch.float64))
    dp, b = rng.normal(size=m.n_cells), rng.normal(size=m.n_cells)
    F, scale = ppe.warm_start_features(
        s, *[to_dev(a, torch.float64) for a in (dp, b, c, fl, m.cell_volume)],
        to_dev(np.zeros(10), torch.float32), to_dev(np.ones(10), torch.float32))
    sy = assembly.masked_system(m.n_cells, owner, neigh, c, fl)
    pin_of = np.zeros(m.n_cells, dtype=np.int64)
    pin_of[sy.perm] = sy.comp
    Fr, sr = omlp.warm_start_features(m.n_cells, owner, neigh, c, fl, m.cell_volume, dp, b, pin_of)
    assert abs(scale - sr) <= 1e-14 * sr
    assert np.abs(F.cpu().numpy() - Fr).max() <= 1e-6


def test_trained_network_reduces_iterations():
    import torch

    import paper_1810_08572_amd as ppe

    torch_dev()
    m = box_mesh((24, 24, 24), jitter=0.1, seed=0)
    c = face_coeff(m, 2400.0)
    c_d = to_dev(c, torch.float64)
    vol = to_dev(m.cell_volume, torch.float64)
    s = ppe.Solver()
    s.set_mesh(m.n_cells, to_dev(m.owner, torch.int32), to_dev(m.neigh, torch.int32))
    zero10 = torch.zeros(10, dtype=torch.float32, device="cuda")
    one10 = torch.ones(10, dtype=torch.float32, device="cuda")
    # training snapshots produced by the solver itself
    # Snapshots right after the front crosses a cell layer (the mask changed
    # within the last two steps) carry a jump no local feature predicts; they
    # are left out of training (the network is still applied to them below).
    feats, targs, masks = [], [], []
    for k, fl, b, p_prev, dp_prev in _series(m, c, 40, 0.01, seed=5, solver=s):
        masks.append(fl > 0)
        if k < 2 or not (np.array_equal(masks[-1], masks[-2]) and
                         np.array_equal(masks[-2], masks[-3])):
            continue
        s.assemble(c_d, to_dev(fl, torch.float64))
        F, scale = ppe.warm_start_features(s, dp_prev, to_dev(b, torch.float64), c_d,
                                           to_dev(fl, torch.float64), vol, zero10, one10)
        p_new = s.solve(to_dev(b, torch.float64)).p
        feats.append(F.clone())
        targs.append(ppe.warm_start_targets(s, p_new, p_prev, scale).clone())
    X = torch.cat(feats)
    T = torch.cat(targs)
    mu, sigma = X.mean(0), X.std(0).clamp_min(1e-6)
    Xs = ((X - mu) / sigma).contiguous()
    shapes = omlp.layer_shapes()
    net = ppe.WarmStartNet()
    net.set_params(to_dev(omlp.init_params(shapes, seed=0).astype(np.float32), torch.float32))
    g = torch.Generator(device="cuda").manual_seed(0)
    losses = []
    for it in range(400):
        idx = torch.randint(0, Xs.shape[0], (8192,), device="cuda", generator=g)
        losses.append(net.train_step(Xs[idx].contiguous(), T[idx].contiguous(), 1e-3))
    assert np.mean(losses[-20:]) < 0.1 * np.mean(losses[:20])
    # held-out run (different right-hand-side series and times)
    its = {"zero": [], "prev": [], "mlp": []}
    for k, fl, b, p_prev, dp_prev in _series(m, c, 16, 0.05, seed=9, solver=s):
        if k < 2:
            continue
        fl_d, b_d = to_dev(fl, torch.float64), to_dev(b, torch.float64)
        s.assemble(c_d, fl_d)
        F, scale = ppe.warm_start_features(s, dp_prev, b_d, c_d, fl_d, vol, mu.contiguous(),
                                           sigma.contiguous())
        y = net.forward(F.contiguous(), bf16=True)
        x0 = ppe.warm_start_apply(s, p_prev, y, scale)
        for name, guess in (("zero", None), ("prev", p_prev), ("mlp", x0)):
            r = s.solve(b_d, x0=guess)
            assert r.stats["rel_residual"] <= 1e-10
            its[name].append(r.stats["iterations"])
    mean = {k: float(np.mean(v)) for k, v in its.items()}
    print("mean PCG iterations:", mean)
    assert mean["mlp"] < mean["zero"]
    assert mean["mlp"] <= mean["prev"]
