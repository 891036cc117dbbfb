"""Pairs whose length ties with min_len: the decision is that of the root of
the sum of rounded squares in the order of the components, whatever the tiles
hold.  Lattice points (many exact ties), and random points with min_len taken
from the pairs themselves, one rounding up and down; FP32 and FP64; a min_len
whose square leaves the range.  Counts are whole numbers: equality."""
import numpy as np
import pytest

import sap_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext, SapError, batch_run  # noqa: E402

DEV = torch.device("cuda:0")


def _lengths(X):
    X = X.astype(np.float64)
    s = np.zeros((len(X), len(X)))
    for l in range(X.shape[1]):
        t = X[:, None, l] - X[None, :, l]
        s = s + t * t
    return np.sqrt(s)[np.triu_indices(len(X), 1)]


def _dropped(X, min_len):
    """Dropped pairs of both forms, and the first minimum of the fused form and
    of the batched engine."""
    Xt = torch.from_numpy(X).to(DEV)
    P0 = torch.from_numpy(sap_inputs.random_orthonormal(np.random.default_rng(1), X.shape[1], 2))
    out = []
    for form in ("fused", "plain"):
        with SapContext(Xt, P0, form=form, min_len=min_len) as ctx:
            out.append(ctx.info()["n_dropped"])
            if form == "fused":
                r = ctx.min_secant()["min_norm"]
    b = batch_run(Xt, [np.arange(len(X), dtype=np.int32)], [dict(set=0, k=2)], [P0.to(DEV)], 1,
                  set_min_len=[min_len])
    return out, r, float(b["min"][0, 0])


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,n", [("lattice", 3), ("random", 7), ("random", 33), ("random", 130)])
def test_ties(kind, n, dtype):
    g = np.random.default_rng(n)
    if kind == "lattice":
        X = (0.1 * g.integers(0, 4, size=(150, n))).astype(dtype)
    else:
        X = g.standard_normal((150, n)).astype(dtype)
    d = _lengths(X)
    kept = np.sort(d[d > 0])
    for q in (0.001, 0.1, 0.5):
        at = kept[int(q * len(kept))]
        for ml in (np.nextafter(at, 0), at, np.nextafter(at, 9)):
            drop, r, rb = _dropped(X, float(ml))
            want = int((d == 0).sum() + ((d > 0) & (d < ml)).sum())
            assert drop == [want, want], (q, ml)
            assert r == rb


def test_range_of_the_square():
    X = np.random.default_rng(0).standard_normal((70, 5))
    drop, r, rb = _dropped(X, 1e-200)
    assert drop == [0, 0] and r == rb
    P0 = torch.from_numpy(sap_inputs.random_orthonormal(np.random.default_rng(1), 5, 2))
    with pytest.raises(SapError, match="NO_PAIRS"):
        SapContext(torch.from_numpy(X).to(DEV), P0, form="fused", min_len=1e200)
