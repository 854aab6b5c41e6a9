"""Warm-start kernels (features, head, FP32 MLP forward / backward, Adam)
against the FP64 oracle (oracle/mlp.py).  The GPU runs the network in fp32
with fp32 accumulation over at most 256 terms per output, so its values and
gradients agree with the FP64 oracle to a relative 1e-4 of the largest
entry (fp32 unit roundoff 6e-8 times the accumulation length, with margin)."""
import numpy as np
import pytest

from oracle import mlp as O

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def dev(x):
    return _torch().from_numpy(np.ascontiguousarray(x)).to("cuda")


def _rows(seed, n):
    rng = np.random.default_rng(seed)
    u = 0.05 * (rng.normal(size=n) + 1j * rng.normal(size=n))
    r = 0.01 * (rng.normal(size=n) + 1j * rng.normal(size=n))
    D = -rng.uniform(1.5, 8.0, size=n)
    t = u + r / D + 0.003 * (rng.normal(size=n) + 1j * rng.normal(size=n))
    u[:3] = 0.0          # zero-amplitude rows (zero-size or symmetry-forbidden pattern)
    return u, r, D, t


def _params(seed, scale=0.1):
    rng = np.random.default_rng(seed)
    return (scale * rng.normal(size=O.n_params())).astype(np.float32)


def test_features_head_step_match_oracle():
    torch = _torch()
    import paper_2004_03682_amd as F
    u, r, D, t = _rows(1, 3001)
    X = torch.empty((u.size, 8), dtype=torch.float32, device="cuda")
    F.ws_features(dev(u), dev(r), dev(D), X)
    x, v, s = O.features(u, r, D)
    assert np.abs(X.cpu().numpy() - x).max() <= 1e-6
    Y = np.random.default_rng(2).normal(size=(u.size, 4)).astype(np.float32)
    out = torch.empty(u.size, dtype=torch.complex128, device="cuda")
    F.ws_apply(dev(Y), dev(u), dev(r), dev(D), out)
    ref = O.predict(Y.astype(np.float64), u, v)
    assert np.abs(out.cpu().numpy() - ref).max() <= 1e-15
    F.ws_apply(None, dev(u), dev(r), dev(D), out)
    assert np.abs(out.cpu().numpy() - (u + v)).max() <= 1e-16
    F.ws_step(dev(u), dev(r), dev(D), out)
    assert np.abs(out.cpu().numpy() - (u + r / D)).max() <= 1e-16
    F.ws_step(None, dev(r), dev(D), out)
    assert np.abs(out.cpu().numpy() - r / D).max() <= 1e-16


def test_forward_matches_oracle():
    torch = _torch()
    import paper_2004_03682_amd as F
    p = _params(3)
    net = F.MLP(seed=0)
    net.set_params(p)
    assert np.array_equal(net.get_params(), p)
    for n in (1, 70, 4099):
        X = np.random.default_rng(n).normal(size=(n, 8)).astype(np.float32)
        Y = torch.empty((n, 4), dtype=torch.float32, device="cuda")
        net.forward(dev(X), Y)
        ref, _ = O.forward(p.astype(np.float64), X.astype(np.float64))
        assert np.abs(Y.cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max(), n
    net.destroy()


@pytest.mark.parametrize("gather,mode", [(False, 0), (True, 0), (False, 1), (True, 1)])
def test_loss_and_gradient_match_oracle(gather, mode):
    torch = _torch()
    import paper_2004_03682_amd as F
    u, r, D, t = _rows(4, 5000)
    p = _params(5)
    net = F.MLP(seed=0)
    net.set_params(p)
    if gather:
        idx = np.random.default_rng(6).choice(u.size, 1777, replace=False)
        L = net.loss_grad(dev(u), dev(r), dev(D), dev(t), idx=dev(idx.astype(np.int64)), mode=mode)
        u, r, D, t = u[idx], r[idx], D[idx], t[idx]
    else:
        L = net.loss_grad(dev(u), dev(r), dev(D), dev(t), mode=mode)
    g = net.get_grad()
    x, v, s = O.features(u, r, D)
    x = x.astype(np.float32).astype(np.float64)        # the network sees fp32 features
    Lo, go = O.loss_and_grad(p.astype(np.float64), x, u, v, t, s, mode)
    assert abs(L - Lo) <= 1e-4 * Lo
    offs = np.cumsum([0] + [int(np.prod(q)) for q in O.SHAPES])
    for k in range(len(O.SHAPES)):
        a, b = g[offs[k]:offs[k + 1]], go[offs[k]:offs[k + 1]]
        assert np.abs(a - b).max() <= 1e-4 * np.abs(go).max() + 1e-4 * np.abs(b).max(), k
    assert np.linalg.norm(g - go) <= 1e-4 * np.linalg.norm(go)
    net.destroy()


def test_adam_steps_match_oracle():
    import paper_2004_03682_amd as F
    u, r, D, t = _rows(7, 2000)
    p = _params(8)
    net = F.MLP(seed=0)
    net.set_params(p)
    q = p.astype(np.float64)
    m = np.zeros_like(q)
    w = np.zeros_like(q)
    for n, lr in ((1, 1e-3), (2, 5e-4), (3, 5e-4)):
        net.loss_grad(dev(u), dev(r), dev(D), dev(t))
        g = net.get_grad().astype(np.float64)
        net.adam(lr)
        q, m, w = O.adam_step(q, g, m, w, n, lr)
        got = net.get_params().astype(np.float64)
        assert np.abs(got - q).max() <= 1e-6 * max(1.0, np.abs(q).max()), n
    net.destroy()


def test_untrained_network_is_the_second_jacobi_iterate_and_training_lowers_the_loss():
    torch = _torch()
    import paper_2004_03682_amd as F
    u, r, D, _ = _rows(9, 20000)
    v = r / D
    t = u + v + (0.3 + 0.05 * D) * v + 0.2j * u     # a learnable correction: a = 0.3 + 0.05 D, b = 0.2 i
    net = F.MLP(seed=11)
    Y = torch.empty((u.size, 4), dtype=torch.float32, device="cuda")
    X = torch.empty((u.size, 8), dtype=torch.float32, device="cuda")
    F.ws_features(dev(u), dev(r), dev(D), X)
    net.forward(X, Y)
    assert torch.count_nonzero(Y).item() == 0
    du, dr, dD, dt = dev(u), dev(r), dev(D), dev(t)
    L0 = net.loss_grad(du, dr, dD, dt)
    for _ in range(200):
        net.loss_grad(du, dr, dD, dt)
        net.adam(1e-3)
    L1 = net.loss_grad(du, dr, dD, dt)
    print("loss", L0, "->", L1, flush=True)
    assert L1 < 0.2 * L0
    net.destroy()


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 127, 129, 8191, 8193])
def test_row_tiles_and_gradient_chunks(rows):
    """Row counts at the edges of the 64-row tiles, of the 32-row gradient slices and of the row chunks
    (128 rows each up to 64 chunks, longer ones above); same bound as above."""
    torch = _torch()
    import paper_2004_03682_amd as F
    u, r, D, t = _rows(rows, rows)
    p = _params(20)
    net = F.MLP(seed=0)
    net.set_params(p)
    L = net.loss_grad(dev(u), dev(r), dev(D), dev(t), mode=1)
    g = net.get_grad()
    x, v, s = O.features(u, r, D)
    x = x.astype(np.float32)
    Lo, go = O.loss_and_grad(p.astype(np.float64), x.astype(np.float64), u, v, t, s, 1)
    assert abs(L - Lo) <= 1e-4 * max(Lo, 1e-30)
    assert np.linalg.norm(g - go) <= 1e-4 * np.linalg.norm(go)
    # the rows past the end of the output stay untouched
    Y = torch.full((rows + 3, 4), 7.0, dtype=torch.float32, device="cuda")
    net.forward(dev(x), Y[:rows])
    ref, _ = O.forward(p.astype(np.float64), x.astype(np.float64))
    got = Y.cpu().numpy()
    assert np.abs(got[:rows] - ref).max() <= 1e-4 * max(np.abs(ref).max(), 1e-30)
    assert (got[rows:] == 7.0).all()
    net.destroy()


@pytest.mark.parametrize("log2n", [5, 13, 17, 19])
def test_bias_gradients_of_large_minibatches(log2n):
    """2^k copies of one row, relative loss: the weight of a row is 2^-k, so in exact arithmetic the gradient is that
    of the single row.  A bias gradient is summed in slices of 32 rows, over the slices of a chunk (1/64 of the rows,
    128 at least) and over the chunks: that many roundings of 2^-24 of the sum of magnitudes at most."""
    _torch()
    import paper_2004_03682_amd as F
    n = 1 << log2n
    u, r, D, t = (x[7:8] for x in _rows(3, 8))
    net = F.MLP(seed=0)
    net.set_params(_params(30))
    net.loss_grad(dev(u), dev(r), dev(D), dev(t), mode=0)
    one = net.get_grad().astype(np.float64)
    net.loss_grad(dev(np.repeat(u, n)), dev(np.repeat(r, n)), dev(np.repeat(D, n)), dev(np.repeat(t, n)), mode=0)
    got = net.get_grad().astype(np.float64)
    per = max(128, n // 64)
    bound = (32 + per // 32 + n // per) * 2.0 ** -24
    b1, b2, b3 = 8 * 256, 8 * 256 + 256 + 256 * 256, 8 * 256 + 256 + 256 * 256 + 256 + 256 * 4
    for at, count in ((b1, 256), (b2, 256), (b3, 4)):
        a, b = got[at:at + count], one[at:at + count]
        assert np.abs(b).max() > 0.0
        assert (np.abs(a - b) <= bound * np.abs(b)).all(), (at, np.abs(a / np.where(b == 0.0, 1.0, b) - 1.0).max())
    net.destroy()


@pytest.mark.parametrize("rows,shift", [(5, 0), (70, 0), (40001, 0), (40001, 32), ((1 << 20) + 77, 0)])
def test_outputs_may_replace_the_inputs(rows, shift):
    """Y in the memory of X (`shift` floats on, within the first row chunk): the same bits as with Y elsewhere."""
    torch = _torch()
    import paper_2004_03682_amd as F
    net = F.MLP(seed=0)
    net.set_params(_params(31))
    X = torch.randn(rows, 8, dtype=torch.float32, device="cuda", generator=torch.Generator("cuda").manual_seed(rows))
    Y = torch.empty(rows, 4, dtype=torch.float32, device="cuda")
    net.forward(X, Y)
    over = X.view(-1)[shift:shift + 4 * rows].view(rows, 4)
    net.forward(X, over)
    assert torch.equal(over, Y)
    net.destroy()
