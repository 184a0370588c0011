"""The network's kernels at the edges of their tiles, against the FP64 oracle.

FP32 products: 32 x 32 and 64 x 64 output tiles, contraction indices in panels
of 64, four values per load where rows are 16-byte aligned.  BF16 inference:
32 columns per workgroup, 32 rows per wave, 256 rows per workgroup, weight
panels of 1024 rows.  Sizes sit on, below and above those, widths are not all
multiples of four, and inputs are also taken from unaligned addresses.

Tolerances as for the full-size network: FP32 forward 1e-5 and gradients 1e-4
relative (Frobenius), BF16 forward 2e-2 (8-bit mantissas).  One Adam step of
lr moves a parameter by at most lr (1 + 1e-3), and where the gradient is above
1e-3 of its maximum by lr sign(g) within 2e-5 (lr = 1e-3).
"""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

# (n_in, n_hidden, n_out, batch)
SHAPES = [(1, 1, 1, 1), (3, 5, 7, 2), (31, 33, 63, 31), (32, 32, 32, 32), (33, 31, 65, 33), (64, 64, 64, 64),
          (65, 100, 130, 65), (128, 96, 260, 255), (40, 72, 36, 257), (60, 1028, 44, 3), (1025, 24, 20, 40),
          (256, 1040, 96, 17)]


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_05194_amd import kpm
    return kpm


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-30))


def _device(a, shift):
    """a on the device, its first element shift floats past an aligned address."""
    import torch
    flat = torch.zeros(a.size + shift, dtype=torch.float32, device="cuda")
    flat[shift:] = torch.tensor(a.ravel(), device="cuda")
    return flat[shift:].view(a.shape)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("scaled", [False, True], ids=["plain", "scaled"])
def test_tile_edges(K, shape, scaled):
    import torch
    n_in, n_hid, n_out, B = shape
    print(f"mlp {shape} scaled={scaled}", flush=True)
    g = np.random.default_rng(n_in * 7 + B)
    net = K.MLP(n_in, n_hid, n_out, seed=2)
    params = [p if p.ndim == 2 else (0.05 * g.normal(size=p.shape)).astype(np.float32) for p in net.get_params()]
    net.set_params(params)
    X = g.normal(size=(B, n_in)).astype(np.float32)
    T = (g.normal(size=(B, n_out)) + 0.3).astype(np.float32)
    w = g.uniform(0.2, 1.0, n_out).astype(np.float32)
    mx, sx, my, sy = (np.zeros(n_in), np.ones(n_in), np.zeros(n_out), np.ones(n_out))
    if scaled:
        Xs, Ts = g.normal(size=(130, n_in)).astype(np.float32), (2.0 * g.normal(size=(130, n_out))).astype(np.float32)
        net.fit_scaling(torch.tensor(Xs, device="cuda"), torch.tensor(Ts, device="cuda"))
        mx, sx, my, sy = Xs.mean(0, np.float64), Xs.std(0, dtype=np.float64), Ts.mean(0, np.float64), Ts.std(0, dtype=np.float64)
    p64 = [p.astype(np.float64) for p in params]
    Yn, cache = omlp.forward(p64, (X.astype(np.float64) - mx) / sx)
    Y = my + sy * Yn
    Tn, wn = (T.astype(np.float64) - my) / sy, w.astype(np.float64) * sy
    G = omlp.backward(p64, cache, Yn, Tn, wn)
    L = omlp.loss(Yn, Tn, wn)
    wd = torch.tensor(w, device="cuda")
    ref_y = None
    for shift in (0, 1):
        xd, td = _device(X, shift), _device(T, shift)
        y = net.forward(xd).cpu().numpy()
        assert rel(y, Y) <= 1e-5
        yb = net.forward(xd, bf16=True).cpu().numpy()
        assert rel(yb, Y) <= 2e-2
        grads, loss = net.gradients(xd, td, wd)
        assert abs(loss - L) <= 1e-5 * L
        for gg, GG in zip(grads, G):
            assert rel(gg, GG) <= 1e-4
        # The alignment decides the loads, not the arithmetic.
        if ref_y is not None:
            assert np.array_equal(y, ref_y[0]) and np.array_equal(yb, ref_y[1])
            assert all(np.array_equal(a, b) for a, b in zip(grads, ref_y[2])) and loss == ref_y[3]
        ref_y = (y, yb, grads, loss)
    # The acceptance measure on the first columns only, after a wider call.
    n_cmp = max(1, n_out // 2)
    ref = Y[:, :n_cmp] + 0.1
    z = net.noise_z(xd, torch.tensor(ref, device="cuda"), torch.full((B,), 1e-2, dtype=torch.float64, device="cuda"),
                    wd[:n_cmp].contiguous(), bf16=True).cpu().numpy()
    d = ref_y[1][:, :n_cmp].astype(np.float64) - ref
    want = np.sqrt(np.sum((w[:n_cmp].astype(np.float64) * d) ** 2, 1)) / (1e-2 * np.sqrt(np.sum(w[:n_cmp].astype(np.float64) ** 2)))
    assert np.max(np.abs(z - want) / want) <= 1e-12
    # One training step: the same loss, and every parameter moved as Adam's first step does.
    loss_d = torch.zeros(1, dtype=torch.float64, device="cuda")
    net.train_step(xd, td, wd, lr=1e-3, loss_out=loss_d)
    assert float(loss_d.item()) == ref_y[3]
    for a, p, gr in zip(net.get_params(), params, G):
        step = a.astype(np.float64) - p
        assert np.max(np.abs(step)) <= 1e-3 * (1 + 1e-3)
        big = np.abs(gr) > 1e-3 * np.max(np.abs(gr))
        want = -1e-3 * gr / (np.abs(gr) + 1e-8)
        assert np.max(np.abs(step - want)[big]) <= 2e-5
    net.close()


def test_column_statistics(K):
    """fit_scaling over row counts around its 64 row groups: forward maps the column mean to 0."""
    import torch
    for n, cols in ((1, 3), (63, 16), (64, 17), (65, 33), (1000, 5)):
        g = np.random.default_rng(n)
        X = (g.normal(size=(n, cols)) * 3.0 + 5.0).astype(np.float32)
        T = (g.normal(size=(n, 2)) * 2.0 - 1.0).astype(np.float32)
        net = K.MLP(cols, 4, 2, seed=1)
        net.fit_scaling(torch.tensor(X, device="cuda"), torch.tensor(T, device="cuda"))
        p64 = [p.astype(np.float64) for p in net.get_params()]
        sx, sy = X.std(0, dtype=np.float64), T.std(0, dtype=np.float64)
        sx[sx == 0] = 1.0
        sy[sy == 0] = 1.0
        Yn, _ = omlp.forward(p64, (X.astype(np.float64) - X.mean(0, np.float64)) / sx)
        y = net.forward(torch.tensor(X, device="cuda")).cpu().numpy()
        assert rel(y, T.mean(0, np.float64) + sy * Yn) <= 1e-5
        net.close()
