"""Window candidates bounded from the unrounded FP64 Y before the exact
evaluations (fused pass, more than four candidates in a block).

Two far points give the set a radius R that makes the FP32 rounding of Y wide
against the spacing of the values, so that a block's window holds many pairs
-- a few, tens, and more than the 256 that are looked at together.  A pair is
left unevaluated only when two others of its block are provably smaller, so
the minimum, its pair, the certificate and the runner-up are what they are
with every candidate evaluated: held against FP64 values of all pairs (the
bars of the parity tests: min within 1e-12 relative plus 2 sqrt(k) n 2^-53,
the same pair unless the runner-up lies within 1e-6)."""
import numpy as np
import pytest

import sap_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapContext  # noqa: E402

DEV = torch.device("cuda:0")


def _values(X, P):
    """Sorted FP64 r of every pair, and the pairs."""
    i, j = np.triu_indices(len(X), 1)
    D = X[i].astype(np.float64) - X[j].astype(np.float64)
    r = np.linalg.norm(D @ P, axis=1) / np.linalg.norm(D, axis=1)
    o = np.lexsort((j, i, r))
    return r[o], i[o], j[o]


@pytest.mark.parametrize("N,n,k,far,dtype", [(517, 20, 1, 1e4, "f32"), (400, 70, 3, 1e6, "f32"), (300, 33, 6, 1e6, "f64"),
                                             (517, 40, 8, 3e6, "f32"), (450, 40, 12, 3e6, "f64"),
                                             (517, 64, 16, 4e6, "f32")])
def test_wide_windows_give_the_fp64_minimum_and_runner_up(N, n, k, far, dtype):
    rng = np.random.default_rng(N + n + k)
    X = rng.standard_normal((N, n))
    X[0], X[1] = far * X[0] / np.linalg.norm(X[0]), -far * X[0] / np.linalg.norm(X[0])
    X = X.astype(np.float32 if dtype == "f32" else np.float64)
    X[5] = X[6]
    X[5, 0] += 1e-3                     # one short pair: the handle then keeps the FP64 Y
    P = sap_inputs.random_orthonormal(rng, n, k)
    with SapContext(torch.from_numpy(X).to(DEV), torch.from_numpy(P), form="fused", close_d=2e-3) as ctx:
        assert ctx.info()["n_close"] == 1
        first = ctx.min_secant()
        for it in range(3):
            P = ctx.get_P().cpu().numpy()
            res = ctx.step()
            r, i, j = _values(X, P)
            tol = 1e-12 * r[0] + 2.0 * np.sqrt(k) * n * 2.0 ** -53
            assert res["certified"] == 1, (it, res)
            assert abs(res["min_norm"] - r[0]) <= tol, (it, res, r[:3])
            assert (res["i"], res["j"]) == (i[0], j[0]) or r[1] - r[0] < 1e-6, (it, res, r[:3])
            if res["runner_up_exact"]:
                assert abs(res["runner_up"] - r[1]) <= tol, (it, res, r[:3])
            else:
                assert res["runner_up"] <= r[1] + tol, (it, res, r[:3])
            inside = int(np.sum(r <= res["coarse_min"] + res["window"]))
            print(f"[cand] N={N} k={k} it {it}: {inside} pairs in the window, {res['n_rescored']} evaluated")
            assert inside > 20, (it, inside, res)    # the data do what they are for
        assert first["min_norm"] > 0.0
    # the run takes the same evaluations
    P0 = sap_inputs.random_orthonormal(rng, n, k)
    with SapContext(torch.from_numpy(X).to(DEV), torch.from_numpy(P0), form="fused", close_d=2e-3) as a, \
            SapContext(torch.from_numpy(X).to(DEV), torch.from_numpy(P0), form="fused", close_d=2e-3) as b:
        tr = a.run(5)
        got = [b.step() for _ in range(5)]
        assert [g["min_norm"] for g in got] == tr["min"].tolist()[:5]
        assert torch.equal(a.get_P(), b.get_P())


def test_more_candidates_than_threads():
    """Every pair of a block inside its window (all r equal at k = n, lists
    full): the first 256 are bounded, the rest evaluated, and the smallest
    pair index wins the tie only if r does -- the value is 1 to rounding."""
    rng = np.random.default_rng(9)
    X = rng.standard_normal((260, 6))
    X[5] = X[6]
    X[5, 0] += 1e-3
    with SapContext(torch.from_numpy(X).to(DEV), torch.eye(6, dtype=torch.float64), form="fused", close_d=2e-3) as ctx:
        res = ctx.min_secant()
    assert abs(res["min_norm"] - 1.0) <= 1e-15 * 8 and res["runner_up"] <= 1.0 + 1e-15
