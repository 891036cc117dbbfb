"""What the bounds from the unrounded Y may strike from a block's window: never
a pair whose 1/d^2 FP32 holds with fewer than 24 bits."""
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
