"""The soft-min is a function of ratios: points scaled by a power of two give
the same loss and the same gradient, bit for bit.  Every quantity of the two
passes then scales exactly (1/d^2 in FP32 by 2^-2e, Y by 2^e, the squares by
2^2e) as long as it stays a normal number, which the scales here leave room
for: the smallest squares are r^2 d^2 2^-100, r about 2^-7.  Masked pairs
(duplicates, the diagonal, the padding) and short pairs are among them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext  # noqa: E402

DEV = torch.device("cuda:0")


def _loss_grad(X, P, tau):
    with SapContext(X, P.cpu(), form="fused") as ctx:
        P32 = P.float().contiguous()
        loss = ctx.softmin_fwd(P32, tau).cpu().numpy()
        return loss, ctx.softmin_bwd(P32, tau, torch.ones(1, device=DEV)).cpu().numpy(), ctx.info()["n_close"]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("k", [3, 7, 10, 16])
def test_loss_and_gradient_do_not_depend_on_the_scale(k, dtype):
    g = torch.Generator().manual_seed(100 + k)
    X = torch.randn(300, 20, generator=g, dtype=torch.float64)
    X[297] = X[5]                             # masked pairs
    X[70] = X[71]
    X[10] = X[11] + 1e-6 * X[12]              # a short pair
    X = X.to(dtype).to(DEV)
    P = torch.linalg.qr(torch.randn(20, k, generator=g, dtype=torch.float64))[0].to(DEV)
    loss, dP, nclose = _loss_grad(X, P, 0.01)
    assert nclose > 0 and np.isfinite(loss[0]) and np.abs(dP).max() > 0.0
    for e in (-50, -44, -30, 40):
        l2, d2, n2 = _loss_grad(X * 2.0 ** e, P, 0.01)
        assert n2 == nclose
        assert np.array_equal(l2, loss), (e, l2, loss)
        assert np.array_equal(d2, dP), (e, np.abs(d2 - dP).max())


@pytest.mark.parametrize("k", [1, 4, 6, 12])
def test_kept_pairs_of_equal_projection_count(k):
    """A kept pair whose projections are equal has r = 0 and its whole weight
    in the sum (a masked one, whose product with 1/d^2 is -0, has none): with
    all r equal to 0, L = -tau log(pairs) in FP32 and the gradient is 0."""
    N, n, tau = 70, 80 + k, 0.25
    X = torch.zeros(N, n, dtype=torch.float64)
    X[torch.arange(N), k + torch.arange(N)] = torch.arange(1, N + 1, dtype=torch.float64)   # off the columns of P
    X[69] = X[68]                                                                            # a duplicate
    P = torch.eye(n, dtype=torch.float64)[:, :k].contiguous()
    loss, dP, _ = _loss_grad(X.to(DEV), P.to(DEV), tau)
    want = -tau * np.log(N * (N - 1) // 2 - 1)
    assert abs(loss[0] - want) <= 2.0 ** -23 * abs(want), (loss, want)
    assert not dP.any()


@pytest.mark.parametrize("k", [1, 10, 16])
def test_column_sums_keep_the_bits_of_two_half_tiles(k):
    """One point's 64 equal terms of the gradient, once on the column side of a
    tile (a sum over the tile's rows in FP32) and, with the points in reverse,
    on the row side (FP64).  The weights are the same bits, so the two
    gradients differ by the rounding of the column sum.  On average it is no
    more than that of two sums of 32 rows, taken on the host for random terms,
    and the roundings of the stored partials and gradients (four of at most u,
    taken as one).  The other points, on a line along the first column of P (r
    near 1, weights below e^-40), make the set large enough for wavefronts that
    hold both halves of a tile."""
    u = 2.0 ** -24
    rng = np.random.default_rng(k)
    f = np.float32
    ref = []
    for c in rng.uniform(1.0, 2.0, 2000).astype(f):
        s = f(0.0)
        for _ in range(32):
            s = f(s + c)
        ref.append(abs(2.0 * float(s) - 64.0 * float(c)) / (64.0 * float(c)))
    N = 8000
    P = torch.eye(65 + k, dtype=torch.float64)[:, :k].contiguous().to(DEV)
    one = torch.ones(1, device=DEV)
    err = []
    for case, h in enumerate(rng.uniform(0.05, 0.4, 64)):
        X = np.zeros((N, 65 + k))
        X[:, 0] = (3.0 + 0.001 * np.arange(N)) * (-1.0) ** np.arange(N)
        X[:64, 0] = h
        X[np.arange(64), k + np.arange(64)] = 1.0    # all at the same distance from the one point
        j = 64 * (1 + case)
        X[j] = 0.0
        X[j, 64 + k] = 1.0                           # a coordinate of its own
        got = []
        for A in (X, np.ascontiguousarray(X[::-1])):
            with SapContext(torch.from_numpy(A).to(DEV), P.cpu(), form="fused", close_d=0.0) as ctx:
                ctx.softmin_fwd(P.float(), 0.01)
                got.append(float(ctx.softmin_bwd(P.float(), 0.01, one)[64 + k, 0]))
        err.append(abs(got[0] - got[1]) / abs(got[1]))
    print(f"[column] k={k}: mean {np.mean(err) / u:.2f} u, max {np.max(err) / u:.2f} u, "
          f"two sums of 32: {np.mean(ref) / u:.2f} u")
    assert np.mean(err) <= np.mean(ref) + u


@pytest.mark.parametrize("tau0", [0.25, 0.8, 1.6])
@pytest.mark.parametrize("k", [2, 8, 16])
def test_gradient_weights_sum_to_one(k, tau0):
    """The weights' exponents use log2(e)/tau rounded to FP32, by 2^-25 to 2^-24
    of it at the tau taken here.  That leaves their sum, and with it the length
    of the gradient, off by at most its part of (max r - min r)/tau; the
    roundings of single pairs (2 million of them) scatter, and are allowed u.
    Times log(pairs) it would be 14 units of the first."""
    u = 2.0 ** -24
    taus = tau0 * (1.0 + np.arange(200) * 1e-3)
    c2 = 1.4426950408889634 / taus
    delta = np.abs(c2.astype(np.float32).astype(np.float64) / c2 - 1.0)
    tau, delta = float(taus[delta.argmax()]), float(delta.max())
    assert delta > 2.0 ** -25
    g = torch.Generator(device=DEV).manual_seed(k)
    X = torch.randn(2000, 40, generator=g, device=DEV, dtype=torch.float64)
    P = torch.linalg.qr(torch.randn(40, k, generator=g, device=DEV, dtype=torch.float64))[0].float()
    with SapContext(X, P.double().cpu(), form="fused") as ctx:
        ctx.softmin_fwd(P, tau)
        got = ctx.softmin_bwd(P, tau, torch.ones(1, device=DEV)).double()
    Y = (X - X.mean(0)) @ P.double()
    d = torch.cdist(X, X, compute_mode="donot_use_mm_for_euclid_dist")
    r = torch.cdist(Y, Y, compute_mode="donot_use_mm_for_euclid_dist") / d
    r.fill_diagonal_(float("inf"))
    rmin, rmax = float(r.min()), float(r[torch.isfinite(r)].max())
    w = torch.exp(-(r - rmin) / tau)
    a = torch.where(torch.isfinite(r), w / (0.5 * w.sum()) / (d * d * r), torch.zeros_like(d))
    want = (X - X.mean(0)).T @ (a.sum(1, keepdim=True) * Y - a @ Y)
    scale = float((got * want).sum() / (want * want).sum() - 1.0)
    print(f"[scale] k={k} tau={tau:.3f}: {scale / u:+.2f} u, rounding of log2(e)/tau {delta / u:.2f} u")
    assert abs(scale) <= delta * (rmax - rmin) / tau + u
