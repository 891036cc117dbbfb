"""The two ways the fused pass reads its y_i rows (staged in LDS, or as scalars),
on both sides of every line of the rule between them: the minimum and its pair
against FP64 values of all pairs, and a run against single steps bit for bit."""
import numpy as np
import pytest

import sap_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext  # noqa: E402

DEV = torch.device("cuda:0")


def _minimum(X, P):
    """Smallest FP64 r over all pairs, and its pair."""
    X, best = X.double(), (float("inf"), -1, -1)
    Y = X @ P
    N = len(X)
    for a in range(0, N, 512):
        d = torch.cdist(X[a:a + 512], X, compute_mode="donot_use_mm_for_euclid_dist")
        c = torch.cdist(Y[a:a + 512], Y, compute_mode="donot_use_mm_for_euclid_dist")
        i = torch.arange(a, min(a + 512, N), device=DEV)
        r = torch.where(i[:, None] < torch.arange(N, device=DEV)[None, :], c / d, torch.full_like(d, 9.0))
        m = int(r.argmin())
        if float(r.view(-1)[m]) < best[0]:
            best = (float(r.view(-1)[m]), a + m // N, m % N)
    return best


@pytest.mark.parametrize("N,k", [
    (65, 1), (130, 4), (300, 7),                         # few blocks: staged
    (2752, 5), (2880, 5),                                # 473 and 518 blocks: two per compute unit
    (4032, 7), (4096, 7), (7040, 3), (7104, 3),          # 1, 1.02, 3.0 and 3.05 items per wavefront
    (130, 8), (1984, 9), (2048, 9), (1984, 15), (2048, 15), (130, 16), (700, 16)])
def test_minimum_on_both_sides_of_the_rule(N, k):
    g = torch.Generator().manual_seed(N + k)
    n = max(12, k + 1)
    X = torch.randn(N, n, generator=g, dtype=torch.float64)
    X = (X.float() if N % 64 else X).to(DEV)
    P0 = torch.from_numpy(sap_inputs.random_orthonormal(np.random.default_rng(k), n, k))
    with SapContext(X, P0, form="fused") as a, SapContext(X, P0, form="fused") as b:
        res = a.min_secant()
        r, i, j = _minimum(X, P0.to(DEV))
        assert res["certified"] == 1 and (res["i"], res["j"]) == (i, j), (res, r, i, j)
        assert abs(res["min_norm"] - r) <= 1e-12 * r + 2.0 * np.sqrt(k) * n * 2.0 ** -53
        tr = b.run(4)
        assert [a.step()["min_norm"] for _ in range(4)] + [a.min_secant()["min_norm"]] == tr["min"].tolist()
        assert torch.equal(a.get_P(), b.get_P())
