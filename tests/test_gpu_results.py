"""What the library reads back from the device: the result of a synchronous
evaluation, the checks of a P, and the soft-min backward's refusal of a P that is not the
forward's, with dP untouched."""
import numpy as np
import pytest

import sap_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import ctypes as C  # noqa: E402

from paper_1807_03425_amd import SapContext, SapError, lib  # noqa: E402

DEV = torch.device("cuda:0")


def _handle(form="fused"):
    w = sap_inputs.make("trig64", N=130, k=5)
    X = torch.from_numpy(w.X).to(DEV)
    return SapContext(X, torch.from_numpy(w.P0), form=form), torch.from_numpy(w.P0).to(DEV)


@pytest.mark.parametrize("form", ["fused", "plain"])
def test_results_interleaved(form):
    """step and min_secant between steps without a result and runs: each
    result is that of its own evaluation, equal to the run's trace."""
    a, P0 = _handle(form)
    b, _ = _handle(form)
    tr = b.run(6)
    mins, ij = tr["min"].cpu().numpy(), tr["ij"].cpu().numpy()
    assert a.min_secant()["min_norm"] == mins[0]
    r = a.step()
    assert r["min_norm"] == mins[0] and [r["i"], r["j"]] == list(ij[0]) and r["t"] >= 0
    a.step(sync=False)
    a.run(1)
    r = a.step()
    assert r["min_norm"] == mins[3] and [r["i"], r["j"]] == list(ij[3])
    assert a.min_secant()["min_norm"] == mins[4]
    a.close()
    b.close()


@pytest.mark.parametrize("bit", [0, 31])
@pytest.mark.parametrize("where", [0, 319, -1])
def test_softmin_refused_P_leaves_dP(where, bit):
    """One flipped bit of P (the sign of a zero included) is refused and
    writes nothing; the backward of the forward's P still works after it."""
    h, P0 = _handle()
    P = P0.float().contiguous()
    P.view(-1)[where] = 0.0
    h.softmin_fwd(P, 0.05)
    one = torch.ones(1, device=DEV)
    want = h.softmin_bwd(P, 0.05, one)
    Q = P.clone()
    Q.view(torch.int32).view(-1)[where] ^= (1 << bit) if bit < 31 else -(1 << 31)
    assert not torch.equal(Q.view(torch.int32), P.view(torch.int32))
    dP = torch.full_like(P, 7.0)
    call = lambda p: lib().sap_softmin_bwd(h.handle, C.c_void_p(p.data_ptr()), 0.05, C.c_void_p(one.data_ptr()),
                                           C.c_void_p(dP.data_ptr()))
    assert call(Q) != 0
    assert bool((dP == 7.0).all())
    torch.cuda.synchronize()
    assert bool((dP == 7.0).all())
    assert call(P) == 0
    torch.cuda.synchronize()
    assert np.array_equal(dP.cpu().numpy(), want.cpu().numpy())
    h.close()


@pytest.mark.parametrize("form", ["fused", "plain"])
@pytest.mark.parametrize("n,k", [(3, 1), (255, 7), (256, 16), (257, 5), (600, 16)])
def test_set_P_checks(n, k, form):
    """Rows around the chunks of 256: a P is taken bit for bit, up to
    |P^T P - I| = 1e-6 in any entry, and a refused one changes nothing."""
    g = np.random.default_rng(n + k)
    X = torch.from_numpy(g.standard_normal((40, n))).to(DEV)
    P0 = np.linalg.qr(g.standard_normal((n, k)))[0]
    h = SapContext(X, torch.from_numpy(P0), form=form)
    P1 = np.linalg.qr(g.standard_normal((n, k)))[0]
    P1[:, -1] *= 1.0 + 0.49e-6                 # squared length within 0.98e-6 of 1
    h.set_P(torch.from_numpy(P1).to(DEV))
    assert np.array_equal(h.get_P().cpu().numpy(), P1)
    ref = h.min_secant()["min_norm"]
    for l in (0, n // 2, n - 1):
        for bad in (np.nan, np.inf, -np.inf):
            Q = P1.copy()
            Q[l, k // 2] = bad
            with pytest.raises(SapError, match="NONFINITE"):
                h.set_P(torch.from_numpy(Q).to(DEV))
    Q = P1.copy()
    Q[:, 0] *= 1.0 + (0.51e-6 if k > 1 else 1e-7)
    if k > 1:
        Q2 = P1.copy()
        Q2[:, 0] += 1.1e-6 * Q2[:, k - 1]      # one product off the diagonal
        refused = [Q, Q2, 1e200 * P1]
    else:
        refused = [1e200 * P1, 0.0 * P1]
    for R in refused:
        with pytest.raises(SapError, match="NOT_ORTHONORMAL"):
            h.set_P(torch.from_numpy(R).to(DEV))
    assert np.array_equal(h.get_P().cpu().numpy(), P1)
    assert h.min_secant()["min_norm"] == ref
    h.close()


def test_P_in_host_memory():
    """set_P and the soft-min read a P in pinned host memory; pageable memory is
    an error."""
    h, P0 = _handle()
    ptr = lambda p: C.c_void_p(p.data_ptr())
    host = torch.empty(P0.shape, dtype=torch.float64, pin_memory=True)
    host.copy_(P0.flip(1))
    assert lib().sap_set_P(h.handle, ptr(host)) == 0
    assert np.array_equal(h.get_P().cpu().numpy(), host.numpy())
    P = P0.float().contiguous()
    h.softmin_fwd(P, 0.05)
    one, dP = torch.ones(1, device=DEV), torch.full_like(P, 7.0)
    want = h.softmin_bwd(P, 0.05, one).cpu().numpy()
    same = torch.empty(P.shape, dtype=torch.float32, pin_memory=True)
    other = torch.empty(P.shape, dtype=torch.float32, pin_memory=True)
    same.copy_(P)
    other.copy_(P)
    other[3, 2] += 0.25
    call = lambda p: lib().sap_softmin_bwd(h.handle, ptr(p), 0.05, ptr(one), ptr(dP))
    assert call(other) != 0 and bool((dP == 7.0).all())
    assert call(same) == 0
    assert np.array_equal(dP.cpu().numpy(), want)
    loss = torch.zeros(1, device=DEV)
    assert lib().sap_softmin_fwd(h.handle, ptr(same), 0.05, ptr(loss)) == 0
    assert call(P) == 0
    assert np.array_equal(dP.cpu().numpy(), want)
    assert lib().sap_set_P(h.handle, ptr(host.clone())) != 0   # (a device error: the handle ends here)
    h.close()
    h, _ = _handle()
    assert lib().sap_softmin_fwd(h.handle, ptr(same.clone()), 0.05, ptr(loss)) != 0
    h.close()


@pytest.mark.parametrize("n,k", [(4800, 1), (700, 3), (257, 7), (40, 16)])
def test_set_P_at_the_tolerance(n, k):
    """Columns whose |P^T P - I| lies within some 1e-16 of 1e-6, above and
    below: accepted exactly where the sum of the rounded products in the order
    of the rows says so."""
    g = np.random.default_rng(n)
    X = torch.from_numpy(g.standard_normal((30, n))).to(DEV)
    P0 = np.linalg.qr(g.standard_normal((n, k)))[0]
    h = SapContext(X, torch.from_numpy(P0), form="fused")
    verdicts = []
    for t in range(-30, 31):
        P = P0.copy()
        P[:, k // 2] *= np.sqrt(1.0 + 1e-6 + 4e-17 * t * (n ** 0.5 / 10.0))
        G = np.array([[np.cumsum(P[:, a] * P[:, b])[-1] for b in range(k)] for a in range(k)])
        want = bool(np.abs(G - np.eye(k)).max() <= 1e-6)
        try:
            h.set_P(torch.from_numpy(P).to(DEV))
            got = True
        except SapError as e:
            assert "NOT_ORTHONORMAL" in str(e)
            got = False
        assert got == want, (t, np.abs(G - np.eye(k)).max() - 1e-6)
        verdicts.append(want)
    assert 5 < sum(verdicts) < 56, sum(verdicts)
    h.close()


def test_set_P_of_long_columns_takes_no_longer():
    """The check's sums are shared by threads: a column of 4800 takes about as
    long as six of 64 (one thread's sum over it took five times as long)."""
    import time
    best = []
    for n, k in ((64, 6), (4800, 1)):
        X = torch.from_numpy(np.random.default_rng(n).standard_normal((30, n))).to(DEV)
        P = torch.from_numpy(np.linalg.qr(np.random.default_rng(k).standard_normal((n, k)))[0])
        with SapContext(X, P, form="fused") as h:
            Pd, t = P.to(DEV), []
            for _ in range(60):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                h.set_P(Pd)
                t.append(time.perf_counter() - t0)
        best.append(min(t))
    print(f"[set_P] {1e6 * best[0]:.0f} us at 64 x 6, {1e6 * best[1]:.0f} at 4800 x 1")
    assert best[1] < 3.0 * best[0]
