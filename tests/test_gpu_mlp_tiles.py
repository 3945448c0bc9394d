"""The combiner's kernels at the edges of their sample tiles (16 and 32) and
of the 256 workgroups a training step runs at most, against float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import paper_2307_04890_amd as tn  # noqa: E402
import tn_inputs as T  # noqa: E402

U = 2.0**-24  # rounding of one FP32 operation
DEPTH = 16 + 64 + 64 + 8  # roundings on the way of one value through the layers


def _layers(p):
    cut = np.cumsum([0, 1024, 64, 4096, 64, 64, 1])
    w1, b1, w2, b2, w3, b3 = (p[a:b] for a, b in zip(cut, cut[1:]))
    return w1.reshape(64, 16), b1, w2.reshape(64, 64), b2, w3.reshape(1, 64), b3


def _data(N, seed):
    """Parameters and N samples none of whose hidden units is within its
    rounding bound of the ReLU's kink."""
    g = np.random.default_rng(seed)
    p = T.mlp_init(seed)
    p += g.normal(0, 0.02, p.shape).astype(np.float32)
    w1, b1, w2, b2, _, _ = (a.astype(np.float64) for a in _layers(p))
    x = -g.random((4 * N + 64, 16), dtype=np.float32) * 5
    z1 = x @ w1.T + b1
    a1 = np.abs(x) @ np.abs(w1).T + np.abs(b1)
    z2 = np.maximum(z1, 0) @ w2.T + b2
    a2 = a1 @ np.abs(w2).T + np.abs(b2)
    clear = (np.abs(z1) > DEPTH * U * a1).all(1) & (np.abs(z2) > DEPTH * U * a2).all(1)
    x = x[clear][:N]
    assert x.shape[0] == N
    return p, np.ascontiguousarray(x), -g.random(N, dtype=np.float32) * 5


def _forward(p, x, absolute=False):
    """Outputs in float64; with absolute the same sums of magnitudes, which
    times DEPTH * U bound the FP32 error."""
    f = np.abs if absolute else (lambda a: a)
    w1, b1, w2, b2, w3, b3 = (f(a.astype(np.float64)) for a in _layers(p))
    x = f(x.astype(np.float64))
    h1 = np.maximum(x @ w1.T + b1, 0)
    h2 = np.maximum(h1 @ w2.T + b2, 0)
    return (h2 @ w3.T + b3)[:, 0], h1, h2


def _unaligned(a):
    """The array on the device, 4 bytes past a 16-byte boundary."""
    buf = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")
    v = buf[1:].view(a.shape)
    v.copy_(torch.from_numpy(a))
    assert v.data_ptr() % 16 == 4 and v.is_contiguous()
    return v


@pytest.mark.parametrize("N", [1, 15, 16, 17, 63, 64, 65, 1000, 32_767, 32_768, 32_769, 65_537])
@pytest.mark.parametrize("aligned", [True, False])
def test_outputs_against_float64(N, aligned):
    # 512 workgroups of four wavefronts hold 32,768 samples at a time
    p, x, _ = _data(N, seed=N)
    dev = (lambda a: torch.from_numpy(a).cuda()) if aligned else _unaligned
    dp, dx = dev(p), dev(x)
    y, _, _ = _forward(p, x)
    bound = DEPTH * U * _forward(p, x, absolute=True)[0]
    got = tn.mlp_forward(dp, dx).cpu().numpy().astype(np.float64)
    assert (np.abs(got - y) <= bound).all()
    n = 100_000
    est = np.random.default_rng(N).integers(1, n, N).astype(np.int32)
    sizes = tn.mlp_predict(dp, dx, n, est=torch.from_numpy(est).cuda()).cpu().numpy().astype(np.float64)
    want = np.minimum(np.maximum(n * np.exp(y), 1), est)
    # the exponential carries the output's error, its own few roundings aside
    assert (np.abs(sizes - want) <= want * (np.expm1(bound) + 8 * U)).all()
    free = tn.mlp_predict(dp, dx, n).cpu().numpy().astype(np.float64)
    want = np.minimum(np.maximum(n * np.exp(y), 1), n)
    assert (np.abs(free - want) <= want * (np.expm1(bound) + 8 * U)).all()


@pytest.mark.parametrize("N", [1, 31, 32, 33, 64, 100, 4096, 8191, 8192, 8193, 16_384])
@pytest.mark.parametrize("aligned", [True, False])
def test_gradient_against_float64(N, aligned):
    # 256 workgroups of 32 samples: past 8192 a workgroup takes several tiles
    p, x, y = _data(N, seed=N + 1)
    idx = np.random.default_rng(N).permutation(N).astype(np.int32)
    dev = (lambda a: torch.from_numpy(a).cuda()) if aligned else _unaligned
    state = [dev(a.copy()) for a in (p, np.zeros_like(p), np.zeros_like(p))]
    dx, dy, di = dev(x), dev(y), torch.from_numpy(idx).cuda()
    loss, grad = tn.mlp_train_step(*state, 1, dx, dy, idx=di, want_grad=True)
    out, h1, h2 = _forward(p, x)
    res = out - y
    w1, b1, w2, b2, w3, b3 = (a.astype(np.float64) for a in _layers(p))

    def gradient(d, h1, h2, m1, m2, f=lambda a: a):
        d2 = d[:, None] * f(w3) * m2
        d1 = (d2 @ f(w2)) * m1
        xs = f(x.astype(np.float64))
        return np.concatenate([(d1.T @ xs).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0),
                               (d[:, None] * h2).sum(0), [d.sum()]])

    m1, m2 = h1 > 0, h2 > 0
    want = gradient(2 * res / N, h1, h2, m1, m2)
    # magnitudes: the residual's own error is the output's bound, and a sum
    # over the samples adds one rounding a term at most
    aout, a1, a2 = _forward(p, x, absolute=True)
    mag = gradient(2 * (np.abs(res) + aout + np.abs(y)) / N, a1, a2, m1, m2, np.abs)
    bound = (2 * DEPTH + N) * U * mag
    assert (np.abs(grad.cpu().numpy() - want) <= bound).all()
    lmag = ((np.abs(res) + aout + np.abs(y)) ** 2).mean()
    assert abs(float(loss) - (res**2).mean()) <= (2 * DEPTH + N) * U * lmag
    # the step without allocation runs the same kernels
    other = [dev(a.copy()) for a in (p, np.zeros_like(p), np.zeros_like(p))]
    l2 = torch.empty(1, device="cuda")
    tn.mlp_train_step_noalloc(*other, 1, dx, dy, idx=di, loss=l2)
    assert all(torch.equal(a, b) for a, b in zip(state, other)) and torch.equal(loss, l2)


@pytest.mark.parametrize("n", [1, 255, 256, 257, 5003])
@pytest.mark.parametrize("aligned", [True, False])
def test_features_against_float64(n, aligned):
    lifted = np.random.default_rng(n).integers(1, n + 1, (16, n)).astype(np.int32)
    d = torch.from_numpy(lifted).cuda()
    x = torch.empty(16 * n + 1, device="cuda")[0 if aligned else 1:][:16 * n]
    ctx = tn.get_context()
    assert tn.lib.tn_mlp_features(ctx.bind_stream(), n, 16, tn.api._dp(d), tn.api._dp(x)) == 0
    want = np.log(lifted.T.astype(np.float64) / n)
    # the ratio's two roundings enter the logarithm as they are; it adds its own
    assert (np.abs(x.view(n, 16).cpu().numpy() - want) <= 3 * U + 4 * U * np.abs(want)).all()


@pytest.mark.parametrize("N", [1, 15, 16, 17, 33, 9000])
def test_rows_off_16_bytes_bounds_and_nan(N):
    # rows that start off 16 bytes take single loads: the same bits; a NaN unit
    # counts as 0 (its layer's other units as they are), and no output passes
    # its node's bound
    p, x = _data(N, seed=71)[:2]
    x[N // 2, 3] = np.nan
    n = 5000
    P = torch.from_numpy(p).cuda()
    est = torch.arange(1, N + 1, dtype=torch.int32, device="cuda")
    got = []
    for lead in (0, 1):
        buf = torch.zeros(16 * N + lead, dtype=torch.float32, device="cuda")
        X = buf[lead:].view(N, 16)
        X.copy_(torch.from_numpy(x))
        got.append((tn.mlp_forward(P, X), tn.mlp_predict(P, X, n), tn.mlp_predict(P, X, n, est=est)))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    y, free, bound = (a.cpu().numpy().reshape(-1) for a in got[0])
    w1, b1, w2, b2, w3, b3 = (a.astype(np.float64) for a in _layers(p))
    h1 = np.fmax(x.astype(np.float64) @ w1.T + b1, 0)
    want = (np.fmax(h1 @ w2.T + b2, 0) @ w3.T + b3)[:, 0]
    clean = np.where(np.isnan(x), 0, x)
    tol = DEPTH * U * _forward(p, clean, absolute=True)[0]
    assert (np.abs(y - want) <= tol).all()
    # (without bounds the outputs stop at n)
    e = est.cpu().numpy()
    assert np.where(free < n, bound == np.minimum(free, e),
                    (bound >= np.minimum(n, e)) & (bound <= e)).all()
