"""Uniform shots at 13 qubits, where the partials are stored past the caches: every row holds the
same counts r, so that the row-averaged coefficient of a Pauli string with support m is the
Walsh sum of r at m over the shots, exactly (a correctly rounded quotient of integers)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1602_08604_amd import lre as L  # noqa: E402

DEV = "cuda:0"


# counts up to hi: partial sums in 32 bits and in binary64
@pytest.mark.parametrize("n,hi", [(12, 3), (13, 3), (13, 40000)])
def test_equal_rows(n, hi):
    print(f"[large uniform n={n} counts <= {hi}]", flush=True)
    d = 2 ** n
    r = np.random.default_rng(n + hi).integers(0, hi + 1, d)
    shots = int(r.sum())
    walsh = r.astype(np.int64)
    for k in range(n):
        walsh = walsh.reshape(-1, 2, 2 ** k)
        walsh = np.stack((walsh[:, 0] + walsh[:, 1], walsh[:, 0] - walsh[:, 1]), 1).reshape(-1)
    counts = torch.empty((3 ** n, d), dtype=torch.uint16, device=DEV)
    counts.view(torch.int16).copy_(torch.from_numpy(r.astype(np.uint16).view(np.int16)).to(DEV).expand(3 ** n, d))
    coef, _ = L.estimate(counts, shots, flags=L.LRE_NO_RHO)
    support = torch.zeros(1, dtype=torch.int64, device=DEV)
    for _ in range(n):                          # letters from the most significant: I or not
        support = (2 * support.unsqueeze(1) + torch.tensor([0, 1, 1, 1], device=DEV)).reshape(-1)
    want = torch.from_numpy(walsh / shots).to(DEV)[support]
    assert torch.equal(coef, want)
