"""The soft-min tile passes against FP64 sums over all pairs at the sizes where
the split of the half-tiles changes: below one half-tile per wavefront, around
one, two and three rounds of blocks, and runs of several half-tiles that begin
and end within a tile or a row of tiles; k of each Y row length, ragged last
tiles, duplicates (masked pairs).

Tolerances as for the coarse evaluation: every r is within e = e_abs + e_rel
of its exact value, so L is within e plus FP32 rounding (about 1e-5 tau, and
2^-24 |L| of the stored loss), and a gradient term, relative, within e / tau
(its weight) plus e / r_min (1/r and y_i - y_j); doubled and quadrupled.  A
lost or doubled half-tile of the smallest set is 1/1056 of the sum.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext  # noqa: E402

DEV = torch.device("cuda:0")


def _reference(X, P, tau):
    X, P = X.double(), P.double()
    Y = (X - X.mean(0)) @ P
    N = X.shape[0]
    rmin, s = None, 0.0
    for rep in range(3):                      # the minimum, the sum, the weights
        Z = torch.zeros_like(Y)
        for a in range(0, N, 256):
            d = torch.cdist(X[a:a + 256], X, compute_mode="donot_use_mm_for_euclid_dist")
            c = torch.cdist(Y[a:a + 256], Y, compute_mode="donot_use_mm_for_euclid_dist")
            keep = d > 0
            r = torch.where(keep, c / d, torch.full_like(d, 1e9))
            if rep == 0:
                rmin = r.min() if rmin is None else torch.minimum(rmin, r.min())
            elif rep == 1:
                s = s + 0.5 * torch.exp(-(r - rmin) / tau).sum()
            else:
                w = torch.where(keep, torch.exp(-(r - L) / tau) / (d * d * r), torch.zeros_like(d))
                Z[a:a + 256] = w.sum(1, keepdim=True) * Y[a:a + 256] - w @ Y
        if rep == 1:
            L = rmin - tau * torch.log(s)
    return float(L), ((X - X.mean(0)).T @ Z), float(rmin)


@pytest.mark.parametrize("N,k", [
    (1984, 3), (2048, 6), (2049, 16),         # 992, 1056, 1122 half-tiles: one round of 1024 wavefronts and more
    (2880, 16), (2881, 10), (2945, 16),       # 2070, 2162: two rounds and more
    (3456, 4), (3520, 12), (3521, 1),         # 2970, 3080, 3192: three rounds and more
    (7013, 10), (7013, 16),                   # 12210: runs of about four (k <= 12) and six
])
def test_softmin_shares(N, k):
    g = torch.Generator(device=DEV).manual_seed(N + k)
    n, tau = 20, 0.05
    X = torch.randn(N, n, generator=g, device=DEV, dtype=torch.float64).float()
    X[N - 3] = X[5]                           # masked pairs: within the set's ends, and one tile
    X[70] = X[71]
    P = torch.linalg.qr(torch.randn(n, k, generator=g, device=DEV, dtype=torch.float64))[0]
    ctx = SapContext(X, P.cpu(), form="fused")
    P32 = P.float()
    loss = ctx.softmin_fwd(P32, tau)
    dP = ctx.softmin_bwd(P32, tau, torch.ones(1, device=DEV))
    L, G, rmin = _reference(X, P32, tau)
    info = ctx.info()
    e = info["e_abs"] + info["e_rel"]
    eL = abs(float(loss) - L)
    eG = float(torch.linalg.norm(dP.double() - G) / torch.linalg.norm(G))
    tL = 2.0 * e + 1e-5 * tau + 2.0 ** -23 * abs(L)
    tG = 4.0 * (e / tau + e / max(rmin, 1e-3)) + 1e-5
    print(f"N={N} k={k} L={L:.6f} errL={eL:.2e} tol={tL:.2e} errG={eG:.2e} tol={tG:.2e} e={e:.1e} rmin={rmin:.1e}")
    assert np.isfinite(eL) and eL <= tL
    assert np.isfinite(eG) and eG <= tG
