"""The learned correction network in every kind of shape: widths on both sides
of the 16-wide fragments and of the 64-wide rows, one layer to eight, batches
on both sides of the 16-sample tiles; against the FP64 oracle."""
import numpy as np
import pytest

gpu = pytest.mark.gpu


def _case(oracle, rng, dims, n):
    """Whole numbers with few weights a row, so that every dot product of the
    forward pass is exact in fp32 in any order (checked): the GPU's layers and
    the oracle's see the same values at every rounding and every ReLU."""
    p = []
    for i in range(len(dims) - 1):
        W = np.zeros((dims[i + 1], dims[i]))
        for o in range(dims[i + 1]):
            at = rng.integers(0, dims[i], 3)
            W[o, at] = rng.choice([-1, 1, 1, 2], 3)
        p += [W.reshape(-1), rng.integers(-3, 4, dims[i + 1])]
    p = np.concatenate(p).astype(np.float64)
    x = rng.integers(-9, 10, (n, dims[0])).astype(np.float64)
    base = rng.integers(0, 30, n).astype(np.float64)
    y, cache = oracle.mlp_forward(p, x, base, dims)
    for ar, Wr, z in cache:
        assert (np.abs(ar) @ np.abs(Wr).T).max() + 3 < 2 ** 24
    assert np.abs(y).max() + 30 < 2 ** 24
    t = y + rng.integers(-40, 41, n)
    return p, x, base, t, y, cache


def _gradient_bound(cache, y, t):
    """Per parameter: the sum over samples of the absolute values of every
    product on the way."""
    dz = np.abs(2.0 * (y - t) / y.size)[:, None]
    out = []
    for li in range(len(cache) - 1, -1, -1):
        ar, Wr, z = cache[li]
        if li < len(cache) - 1:
            dz = dz * (z > 0)
        out += [dz.sum(0), (dz.T @ np.abs(ar)).reshape(-1)]
        dz = dz @ np.abs(Wr)
    return np.concatenate(out[::-1])


@gpu
@pytest.mark.parametrize("n", [1, 17, 200])
@pytest.mark.parametrize("n_in,hidden,layers", [
    (1, 1, 1), (64, 64, 7), (16, 16, 3), (17, 15, 2), (33, 48, 1), (5, 63, 7),
    (64, 1, 2), (1, 64, 4), (15, 17, 5), (20, 49, 3), (48, 33, 6)])
def test_shapes(oracle, n_in, hidden, layers, n):
    """Forward values exactly; each gradient element within 2^-13 of the
    absolute contraction (paths of at most 8 * 64 + 200 / 8 + 8 < 2^10.1
    roundings of 2^-24, and the loss terms' own); after Adam steps the weight
    images are those of a network created from the same parameters."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(n_in * 1000 + hidden * 10 + layers + n)
    dims = (n_in,) + (hidden,) * layers + (1,)
    print("[case] mlp shape", dims, "n", n, flush=True)
    p, x, base, t, y_ref, cache = _case(oracle, rng, dims, n)
    f32 = lambda a: torch.from_numpy(np.asarray(a, np.float32)).cuda()
    m = C.MLP(p.astype(np.float32), n_in, hidden, layers)
    xd, bd, td = f32(x), f32(base), f32(t)
    y = m.forward(xd, bd)
    loss = m.train_step(xd, bd, td, lr=0.0)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().astype(np.float64), y_ref)
    l_ref, g_ref = oracle.mlp_loss_grad(p, x, base, t, dims)
    assert abs(loss.item() - l_ref) <= 2.0 ** -20 * max(1.0, l_ref)
    g = m.read(1).astype(np.float64)
    G = _gradient_bound(cache, y_ref, t)
    assert np.all(np.abs(g - g_ref) <= 2.0 ** -13 * G)
    for _ in range(3):
        m.train_step(xd, bd, td, lr=1e-3)
    other = C.MLP(m.read(0), n_in, hidden, layers)
    a, b = m.forward(xd, bd), other.forward(xd, bd)
    la = m.train_step(xd, bd, td, lr=0.0).clone()
    lb = other.train_step(xd, bd, td, lr=0.0)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert torch.equal(la.view(torch.int32), lb.view(torch.int32))
    assert np.array_equal(m.read(1), other.read(1))
    m.close()
    other.close()


@gpu
@pytest.mark.parametrize("n_in,hidden,layers", [(5, 63, 7), (17, 15, 2)])
def test_infinite_inputs_stay_with_their_sample(n_in, hidden, layers):
    """An infinite or NaN input changes its own sample's output only."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2102_02440_amd import compass as C
    rng = np.random.default_rng(hidden)
    n = 37
    m = C.MLP(rng.normal(size=C.mlp_n_params(n_in, hidden, layers)).astype(np.float32) * 0.3,
              n_in, hidden, layers)
    print("[case] mlp infinite", n_in, hidden, layers, flush=True)
    x = rng.normal(size=(n, n_in)).astype(np.float32)
    base = torch.zeros(n, device="cuda")
    ref = m.forward(torch.from_numpy(x).cuda(), base).cpu().numpy()
    bad = x.copy()
    bad[3, 0], bad[20, n_in - 1], bad[36, 2] = np.inf, -np.inf, np.nan
    got = m.forward(torch.from_numpy(bad).cuda(), base).cpu().numpy()
    keep = np.ones(n, bool)
    keep[[3, 20, 36]] = False
    assert np.array_equal(got[keep], ref[keep]) and np.isfinite(got[keep]).all()
    m.close()
