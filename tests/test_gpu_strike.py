"""What the bounds from the unrounded Y may strike from a block's window: more
candidates than are looked at together, the smallest pair among those that are
not, and 1/d^2 that FP32 holds with fewer than 24 bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext  # noqa: E402

DEV = torch.device("cuda:0")


def _values(X, P):
    """Sorted FP64 r of every pair, and the pairs."""
    i, j = np.triu_indices(len(X), 1)
    D = X[i] - X[j]
    r = np.linalg.norm(D @ P, axis=1) / np.linalg.norm(D, axis=1)
    o = np.lexsort((j, i, r))
    return r[o], i[o], j[o]


def _late_minimum(k, seed):
    """64 points (one tile, one block; k >= 8: a list per 16 rows) with some 350
    pairs of distinct r in the window, 70 to 120 in each list, the smallest the
    last pair of all.  27 points differ little in the plane of P, the others
    much; two far points make the window wide, one short pair (r = 1) makes the
    handle keep the FP64 Y."""
    rng = np.random.default_rng(seed)
    n = 40
    P = np.linalg.qr(rng.standard_normal((n, n)))[0]
    P, Q = P[:, :k], P[:, k:]
    special = np.zeros(64, bool)
    for q, m in enumerate((5, 4, 5, 13)):
        special[16 * q + 16 - m:16 * q + 16] = True
    A, B = rng.standard_normal((64, k)), rng.standard_normal((64, n - k))
    A /= np.linalg.norm(A, axis=1, keepdims=True)
    B /= np.linalg.norm(B, axis=1, keepdims=True)
    X = np.where(special[:, None], A @ P.T + 3.3 * B @ Q.T, 12.0 * A @ P.T + B @ Q.T)
    mid, t = 0.5 * (X[62] + X[63]) @ P, (X[62] - X[63]) @ P
    for p, s in ((62, 0.3), (63, -0.3)):
        X[p] += (mid + s * t / np.linalg.norm(t) - X[p] @ P) @ P.T
    f = rng.standard_normal(n)
    f /= np.linalg.norm(f)
    X[0], X[1] = 4e6 * f, -4e6 * f
    X[3] = X[2] + 1e-3 * P[:, 0]
    return X, np.ascontiguousarray(P)


@pytest.mark.parametrize("k,seed", [(8, 1), (12, 0), (16, 0)])
def test_more_than_256_candidates_with_the_smallest_last(k, seed):
    X, P = _late_minimum(k, seed)
    r, i, j = _values(X, P)
    assert (i[0], j[0]) == (62, 63) and r[1] - r[0] > 1e-3 and r[2] - r[1] > 1e-6
    with SapContext(torch.from_numpy(X).to(DEV), torch.from_numpy(P), form="fused", close_d=2e-3) as ctx:
        assert ctx.info()["n_close"] == 1
        res = ctx.min_secant()
    tol = 1e-12 * r[0] + 2.0 * np.sqrt(k) * 40 * 2.0 ** -53
    inside = int(np.sum(r <= res["coarse_min"] + res["window"]))
    print(f"[strike] k={k}: {inside} pairs in the window, {res['n_rescored']} evaluated")
    assert res["certified"] == 1 and (res["i"], res["j"]) == (62, 63), res
    assert abs(res["min_norm"] - r[0]) <= tol
    assert res["runner_up_exact"] == 1 and abs(res["runner_up"] - r[1]) <= tol, (res, r[:3])
    assert inside > 256 + 20 and inside - 256 < res["n_rescored"] < inside // 2, (inside, res)


@pytest.mark.parametrize("shift", [0, -40])
def test_subnormal_inverse_lengths_strike_nothing(shift):
    """Six pairs inside one window whose 1/d^2 near 2^-134 are FP32 subnormals:
    five are held exactly, that of the smallest r is rounded up by nearly 2^-16,
    which puts the r its bounds would start from above two of the others.  At
    2^-40 times the size all are normal numbers, and the same pair comes out."""
    r0, d2 = 2.0 ** -5, 2.0 ** 134
    w = (2.0 ** 15 + 0.502) * 2.0 ** -149            # rounds up to the next subnormal
    N = 14
    X = np.zeros((N, 9))
    pairs = [(d2, 1.0 + 1e-7), (d2, 1.0 + 1e-5), (1.0 / w, 1.0 - 3e-6), (d2, 1.0 + 1.1e-5), (d2, 1.0),
             (d2, 1.0 + 1.2e-5)]
    for m, ((dd, f), c) in enumerate(zip(pairs, (-3, -2, -1, 1, 2, 3))):
        dy = r0 * f * np.sqrt(dd)
        half = 0.5 * np.array([dy, np.sqrt(dd - dy * dy)])
        for s, row in ((1.0, 2 * m), (-1.0, 2 * m + 1)):
            X[row, 0] = c * 2.0 ** 66 + s * half[0]
            X[row, 1 + m] = s * half[1]
    X[12, 8], X[13, 8] = 2.0 ** 59, -2.0 ** 59       # one short pair: the handle then keeps the FP64 Y
    P = np.eye(9)[:, :1].copy()
    r, i, j = _values(X, P)
    r, i, j = r[1:], i[1:], j[1:]                    # (the short pair's r is 0)
    assert (i[0], j[0]) == (4, 5) and r[1] - r[0] > 2e-6 * r[0]
    X[12, 0] = 2.0 ** 59                             # now about 1/2
    with SapContext(torch.from_numpy(X * 2.0 ** shift).to(DEV), torch.from_numpy(P), form="fused",
                    close_d=2.0 ** (62 + shift)) as ctx:
        assert ctx.info()["n_close"] == 1
        res = ctx.min_secant()
    assert res["certified"] == 1 and (res["i"], res["j"]) == (4, 5), (res, r[:7], i[:7])
    assert abs(res["min_norm"] - r[0]) <= 1e-12 * r[0] + 18.0 * 2.0 ** -53
