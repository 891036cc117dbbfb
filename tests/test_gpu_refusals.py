"""What a refused call leaves behind and costs."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1807_03425_amd import SapError, batch_run  # noqa: E402

DEV = torch.device("cuda:0")


class _Mallinfo2(C.Structure):
    _fields_ = [(f, C.c_size_t) for f in ("arena", "ordblks", "smblks", "hblks", "hblkhd", "usmblks", "fsmblks",
                                          "uordblks", "fordblks", "keepcost")]


@pytest.mark.parametrize("what", ["start", "X"])
def test_refused_batches_leave_no_host_memory(what):
    """Batches refused for a start that is not orthonormal, or for a NaN in X,
    with stats asked for: no event stays behind (three of at least 100 bytes
    per call would be 900 KB after 3000 calls; allowed are 100 KB)."""
    libc = C.CDLL(None)
    libc.mallinfo2.restype = _Mallinfo2
    X = torch.from_numpy(np.random.default_rng(1).standard_normal((60, 8))).to(DEV)
    if what == "X":
        X[3, 2] = float("nan")
    P0 = [(2.0 if what == "start" else 1.0) * np.eye(8)[:, :2]]

    def refuse(times):
        for _ in range(times):
            try:
                batch_run(X, [np.arange(40)], [dict(set=0, k=2)], P0, 1)
            except SapError:
                continue
            raise AssertionError("accepted")
        return libc.mallinfo2().uordblks

    before = refuse(500)
    after = refuse(3000)
    print(f"[leak] {what}: {(after - before) / 3000:.1f} bytes per refused call")
    assert after - before < 100_000
