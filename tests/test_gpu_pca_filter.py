"""The secant-PCA start where its filter's form changes: one block for n <= 64
and for n <= 128 with at most 16 vectors, launches above.  Against the
oracle's explicit SVD; graded points, so that the span is well defined.  The
start stops at a residual of 1e-12 of the largest eigenvalue, and eigenvalues
k and k + 1 are at least 0.02 of it apart: the span is within 1e-12 / 0.02 of
the exact one, 1e-10 with rounding."""
import numpy as np
import pytest

import oracle
import sap_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("N,n,k", [(90, 16, 3), (90, 63, 4), (90, 64, 8), (90, 64, 9), (140, 65, 8), (140, 65, 9),
                                   (140, 100, 1), (140, 128, 8), (140, 128, 9), (140, 129, 8)])
def test_filter_forms(N, n, k):
    g = np.random.default_rng(n + k)
    X = g.standard_normal((N, n)) * 0.85 ** np.arange(n)
    P0 = sap_inputs.random_orthonormal(g, n, k)
    with SapContext(torch.from_numpy(X).to(DEV), torch.from_numpy(P0), form="fused") as ctx:
        P, info = ctx.pca_init()
    P = P.cpu().numpy()
    Po, sv, every = oracle.pca_init(X, k)
    assert every[k - 1] ** 2 - every[k] ** 2 >= 0.02 * every[0] ** 2
    assert info["converged"] == 1
    assert np.abs(P @ P.T - Po @ Po.T).max() <= 1e-10
    assert np.max(np.abs(np.array(info["sigma"]) - sv) / sv) <= 1e-11
