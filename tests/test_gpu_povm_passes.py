"""The reduced measurement set at the sizes where its passes change: 7 digits in the first
pass (n = 7 alone, n >= 11), 6 + register passes (n = 9), 7 + 5 (n = 12), three passes
(n = 13); empty data and a singular operator set are reported from every form.

Bar for the sampled coefficients: 64 n 2^-53 times the scale of the coefficient's terms, as
n mode products of four-term sums and one division round; counts near the uint16 limit
make every partial sum as large as it can get.
"""
import numpy as np
import pytest

import oracle
from tests.test_gpu_povm import tetra_G

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1602_08604_amd import lre as L  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("n", [6, 7, 9, 11, 12, 13])
def test_povm_passes(n):
    print(f"[povm passes n={n}]", flush=True)
    rng = np.random.default_rng(300 + n)
    c = rng.integers(65000, 65536, size=4 ** n).astype(np.uint16)
    c[rng.integers(0, 4 ** n, 4 ** n // 3)] = 0
    G = tetra_G()
    coef, _ = L.povm_estimate(torch.from_numpy(c).to(DEV), G, flags=L.LRE_NO_RHO)
    e = coef.cpu().numpy()
    # the ends, one index per digit value and position, and random ones
    idx = np.unique(np.concatenate([[0, 4 ** n - 1], [a << (2 * k) for a in (1, 2, 3) for k in range(n)],
                                    rng.integers(0, 4 ** n, 24)]))
    ref, cond = oracle.povm_coefs_direct(n, c, G, idx)
    dev = np.abs(e[idx] - ref)
    print(f"[povm n={n}: max dev {dev.max():.2e}]", flush=True)
    assert np.all(dev <= 64 * n * 2.0 ** -53 * cond)


@pytest.mark.parametrize("n", [5, 6, 7, 8, 9, 12])
def test_povm_reports(n):
    print(f"[povm reports n={n}]", flush=True)
    G = tetra_G()
    z = torch.zeros(4 ** n, dtype=torch.uint16, device=DEV)
    with pytest.raises(L.LreError) as err:
        L.povm_estimate(z, G, flags=L.LRE_NO_RHO)
    assert err.value.status == L.LRE_E_EMPTY_BASIS
    one = z.clone()
    one[-1:] = torch.ones(1, dtype=torch.uint16, device=DEV)
    bad = G.copy()
    bad[:, 2] = bad[:, 1]
    with pytest.raises(L.LreError) as err:
        L.povm_estimate(one, bad, flags=L.LRE_NO_RHO)
    assert err.value.status == L.LRE_E_ARG
    coef, _ = L.povm_estimate(one, G, flags=L.LRE_NO_RHO)       # one count is not empty
    assert abs(coef[0].item() - 1) <= 1e-12
