"""The precomputed 1/d^2 tiles (staged 32 components at a time, 4 x 4 pairs
per thread) at the edges of their chunks and tiles: component counts around
multiples of 32, point counts around multiples of 64, rows longer than n,
FP32 and FP64 points, duplicates and a length threshold.

The oracle counts the kept and dropped pairs and gives the minimum.  The
handle's minimum is an FP64 evaluation from X whatever the tiles hold, so the
tiles themselves are checked through their consumer of every pair, the
soft-min loss at a large tau (there L = -tau log(pairs) + mean r to first
order: every pair counts alike), against the same sum in FP64.  r is the
coarse value, |r~ - r| <= e_abs + e_rel r, and the loss is a weighted mean of
the r, so |dL| <= e_abs + e_rel plus the FP32 rounding of exp2 and of the
sums (32 terms: under 36 2^-24, 2^-18 tau covers it) and of the returned
loss."""
import numpy as np
import pytest

import oracle
import sap_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext, SapError  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,n,pad,min_len", [(2, 1, 0, 0.0), (63, 31, 1, 0.0), (64, 32, 0, 1.0), (65, 33, 3, 0.0),
                                             (129, 64, 0, 0.0), (130, 65, 2, 2.0), (200, 97, 0, 0.0)])
def test_tiles_at_chunk_and_tile_edges(dtype, N, n, pad, min_len):
    rng = np.random.default_rng(1000 * N + n)
    X = rng.standard_normal((N, n)).astype(np.float32 if dtype == "f32" else np.float64)
    if N > 20:
        X[7] = X[3]
        X[N - 1] = X[3]
    k = min(n, 3)
    P0 = sap_inputs.random_orthonormal(rng, n, k)
    buf = torch.full((N, n + pad), float("nan"), dtype=torch.float32 if dtype == "f32" else torch.float64, device=DEV)
    buf[:, :n] = torch.from_numpy(X).to(DEV)
    ref = oracle.min_secant(X, P0, min_len=min_len)
    with SapContext(buf[:, :n], torch.from_numpy(P0), form="fused", min_len=min_len) as ctx:
        info = ctx.info()
        assert info["n_pairs"] == ref["n_pairs"] and info["n_dropped"] == N * (N - 1) // 2 - ref["n_pairs"]
        r = ctx.min_secant()
        assert (r["i"], r["j"]) == (ref["i"], ref["j"]) or ref["r_second"] - ref["r_min"] < 1e-6
        assert abs(r["min_norm"] - ref["r_min"]) <= 1e-12 * ref["r_min"] + 2.0 * np.sqrt(k) * n * 2.0 ** -53
        tau = 5.0
        P32 = torch.from_numpy(P0.astype(np.float32)).to(DEV)
        L = float(ctx.softmin_fwd(P32, tau).item())
    want = oracle.softmin(X, P0.astype(np.float32).astype(np.float64), tau, min_len=min_len)["L"]
    tol = info["e_abs"] + info["e_rel"] + tau * 2.0 ** -18 + abs(want) * 2.0 ** -23
    assert abs(L - want) <= tol, (L, want, tol)


@pytest.mark.parametrize("form", ["plain", "fused"])
@pytest.mark.parametrize("N,n", [(2, 3), (20, 7), (600, 9)])   # plain: a secant array below and above 1 MB
def test_refused_points(N, n, form):
    """NaN and Inf in X, every pair a duplicate, and both: the same refusals
    whether or not the secants are built before X is known to be finite."""
    g = np.random.default_rng(N)
    good = g.standard_normal((N, n))
    P = torch.from_numpy(np.linalg.qr(g.standard_normal((n, 2)))[0])

    def refused(X):
        try:
            SapContext(torch.from_numpy(X).to(DEV), P, form=form).close()
        except SapError as e:
            return str(e).split(":")[0]
    for bad in (np.nan, np.inf, -np.inf):
        X = good.copy()
        X[N - 1, n - 1] = bad
        assert refused(X) == "SAP_ERR_NONFINITE"
    same = np.repeat(good[:1], N, axis=0)
    assert refused(same) == "SAP_ERR_NO_PAIRS"
    same[0, 0] = np.nan
    assert refused(same) == "SAP_ERR_NONFINITE"
    assert refused(good) is None
