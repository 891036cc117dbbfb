"""1/d^2 tiles at the edges of the staged chunk of 16 components (n = 15, 16,
17 and around 32): the minimum and its pair against FP64 values of all pairs,
in the fused form and in the batched engine, and sigma of the secant-PCA start."""
import numpy as np
import pytest

import sap_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext, batch_run  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 32, 33])
def test_distances_at_chunk_edges(n, dtype):
    rng = np.random.default_rng(n)
    k = min(n - 1, 3)
    X = rng.standard_normal((130, n)).astype(dtype)
    P = sap_inputs.random_orthonormal(rng, n, k)
    i, j = np.triu_indices(130, 1)
    D = X[i].astype(np.float64) - X[j].astype(np.float64)
    d = np.linalg.norm(D, axis=1)
    r = np.linalg.norm(D @ P, axis=1) / d
    tol = 1e-12 * r.min() + 2.0 * np.sqrt(k) * n * 2.0 ** -53
    Xt = torch.from_numpy(X).to(DEV)
    with SapContext(Xt, torch.from_numpy(P), form="fused") as ctx:
        res = ctx.min_secant()
        sigma = np.array(ctx.pca_init()[1]["sigma"])
    assert res["certified"] == 1 and abs(res["min_norm"] - r.min()) <= tol
    out = batch_run(Xt, [np.arange(130)], [dict(set=0, k=k)], [P], 0)
    assert int(out["certified"][0, 0]) == 1 and abs(float(out["min"][0, 0]) - r.min()) <= tol
    S = D / d[:, None]
    want = np.sqrt(np.linalg.eigvalsh(S.T @ S)[::-1][:k])
    assert np.allclose(sigma, want, rtol=1e-11, atol=0.0), (sigma, want)
