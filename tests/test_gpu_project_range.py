"""Step (iii) of 7 and 8 qubits on entries near the ends of the type's range, where squares of
entries under- or overflow: small amplitudes, one tiny coherence, the whole matrix scaled by
a power of two.

Tolerance: as for the other spectra, eigenvalues within c d eps |mu| and rho within sqrt(d)
times that: 1e-12 and 1e-11 at d <= 256, |mu| <= 1 (of the matrix before it is scaled)."""
import numpy as np
import pytest

from oracle import project as OP

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1602_08604_amd import lre as L  # noqa: E402
from tests.test_gpu_project_forms import _matrix  # noqa: E402

DEV = "cuda:0"


def _check(r, scale=1.0):
    ref, m, _ = OP.project(r)
    rho, ev = L.project(torch.from_numpy(r * scale).to(DEV))
    assert np.max(np.abs(ev.cpu().numpy() / scale - m)) <= 1e-12
    assert np.max(np.abs(rho.cpu().numpy() / scale - ref)) <= 1e-11


@pytest.mark.parametrize("amplitude", [1e-12, 1e-20, 1e-40])
@pytest.mark.parametrize("n", [7, 8])
def test_small_amplitudes(n, amplitude):
    """A product state of (1, amplitude) per qubit: entries down to amplitude^(2 n)."""
    print(f"[project range n={n} amplitude {amplitude}]", flush=True)
    psi = np.ones(1, dtype=np.complex128)
    for k in range(n):
        psi = np.kron(psi, np.array([1.0, amplitude * 1j ** k]))
    _check(np.outer(psi, psi.conj()))


@pytest.mark.parametrize("entry", [1e-170j, 3e-161 + 1e-165j, 1e-320])
@pytest.mark.parametrize("n", [7, 8])
def test_tiny_coherence(n, entry):
    print(f"[project range n={n} coherence {entry}]", flush=True)
    r = _matrix("diagonal", n)
    for i, j in ((1, 0), (2 ** n - 1, 2 ** n - 2), (2 ** n - 1, 3)):
        r[i, j], r[j, i] = entry, np.conj(entry)
    _check(r)


@pytest.mark.parametrize("scale", [2.0 ** -600, 2.0 ** -90, 2.0 ** 110, 2.0 ** 600])
@pytest.mark.parametrize("n", [7, 8])
def test_scale(n, scale):
    print(f"[project range n={n} scale {scale}]", flush=True)
    _check(_matrix("dense", n), scale)
