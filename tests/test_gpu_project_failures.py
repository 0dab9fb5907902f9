"""Step (iii) where there is no result: LRE_E_EIG through lre_check and rho = 0, never NaN with a
good status.  7 and 8 qubits: input that is not finite anywhere in the triangle that is read.
9 qubits (the library's solver): a diagonal matrix, whose back-transformation may give NaN."""
import numpy as np
import pytest

from oracle import project as OP

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1602_08604_amd import lre as L  # noqa: E402
from tests.test_gpu_project_forms import _matrix  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("value", [np.nan, np.inf, complex(0, -np.inf), 1e308])
@pytest.mark.parametrize("n", [5, 7, 8])
def test_not_finite(n, value):
    """(1e308 in a whole row and column: finite, but its norm is not.)"""
    d = 2 ** n
    for i, j in ((d - 1, 0), (d // 2, 5), (d - 1, d - 1)):
        print(f"[project failure n={n} {value} at {i}, {j}]", flush=True)
        if i == j and isinstance(value, complex):
            continue                               # (the diagonal's imaginary part is not read)
        r = _matrix("dense", n)
        if value == 1e308:
            if n == 5:
                continue                           # (the one-workgroup form scales its input)
            r[i, :] = r[:, i] = value
        r[i, j], r[j, i] = value, np.conj(value)
        rho = torch.full((d, d), 7.0, dtype=torch.complex128, device=DEV)
        with pytest.raises(L.LreError) as e:
            L.project(torch.from_numpy(r).to(DEV), rho=rho)
        assert e.value.status == L.LRE_E_EIG
        assert not rho.any().item()
    rho, _ = L.project(torch.from_numpy(_matrix("dense", n)).to(DEV))      # and the next call is well
    assert np.max(np.abs(rho.cpu().numpy() - OP.project(_matrix("dense", n))[0])) <= 1e-11


@pytest.mark.parametrize("kind", ["diagonal", "identity"])
def test_library_result_is_checked(kind):
    n = 9
    print(f"[project failure n={n} {kind}]", flush=True)
    r = _matrix(kind, n)
    rho = torch.full(r.shape, 7.0, dtype=torch.complex128, device=DEV)
    try:
        L.project(torch.from_numpy(r).to(DEV), rho=rho)
    except L.LreError as e:
        assert e.status == L.LRE_E_EIG
        assert not rho.any().item()
    else:
        assert np.max(np.abs(rho.cpu().numpy() - OP.project(r)[0])) <= 1e-11
