"""The last pass and step (ii) in one launch (6 to 8 qubits) against the two passes by
themselves: coefficients as without a matrix, the matrix as eq. (4) of those coefficients.

Uniform shots: the same integers and correctly rounded quotients, so equality.  Per-basis
totals: the folds add the same at most 6^(n-5) values in another order, some 8 n 2^-53 of
their mean magnitude (at most 1): 1e-13.  mu: within 1e-12 of the oracle, exactly Hermitian.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1602_08604_amd import lre as L  # noqa: E402
from tests.test_gpu_tiles import as_uint16, uniform_counts  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("hi", [9, 65535])       # sums in 32 bits, and beyond them
@pytest.mark.parametrize("n", [6, 7, 8])
def test_uniform(n, hi, fp32):
    print(f"[fused rho n={n} counts <= {hi} fp32={fp32}]", flush=True)
    c, shots = uniform_counts(n, hi, 900 + n)
    c = as_uint16(c)
    want, _ = L.estimate(c, shots, flags=L.LRE_NO_RHO)
    coef, rho = L.estimate(c, shots, flags=L.LRE_RHO_FP32 if fp32 else 0)
    assert torch.equal(coef, want)
    mu = rho.cpu().numpy()
    assert np.max(np.abs(mu - oracle.rho(n, coef.cpu().numpy()))) <= (1e-6 if fp32 else 1e-12)
    assert np.array_equal(mu, mu.conj().T)


@pytest.mark.parametrize("given", [True, False])
@pytest.mark.parametrize("n", [6, 7, 8])
def test_per_basis(n, given):
    print(f"[fused rho per-basis n={n} given={given}]", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(40 + n)
    c = torch.randint(0, 200, (3 ** n, 2 ** n), generator=g, device=DEV)
    nb = c.sum(1).to(torch.int32) if given else None
    c = as_uint16(c)
    want, _ = L.estimate(c, 0, n_per_basis=nb, flags=L.LRE_NO_RHO)
    coef, rho = L.estimate(c, 0, n_per_basis=nb)
    assert (coef - want).abs().max().item() <= 1e-13
    mu = rho.cpu().numpy()
    assert np.max(np.abs(mu - oracle.rho(n, coef.cpu().numpy()))) <= 1e-12
    assert np.array_equal(mu, mu.conj().T)


@pytest.mark.parametrize("n", [6, 7, 8])
def test_row_check(n):
    """A wrong row anywhere is reported by the launch that also makes the matrix."""
    c, shots = uniform_counts(n, 9, 70 + n)
    for row in (0, 3 ** n // 2, 3 ** n - 1):
        print(f"[fused rho row check n={n} row={row}]", flush=True)
        d = c.clone()
        d[row, 3] += 1
        with pytest.raises(L.LreError) as e:
            L.estimate(as_uint16(d), shots)
        assert e.value.status == L.LRE_E_SHOTS
