"""Step (iii) adds in a fixed order: repeated calls on one input give the same bits."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1602_08604_amd import lre as L  # noqa: E402
from tests.test_gpu_project_forms import _matrix  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("n", [3, 5, 6, 7, 8])
@pytest.mark.parametrize("kind", ["dense", "graded"])
def test_same_bits(n, kind):
    print(f"[project repeat n={n} {kind}]", flush=True)
    mu = torch.from_numpy(_matrix(kind, n)).to(DEV)
    rho, ev = L.project(mu)
    for _ in range(20):
        again, ev2 = L.project(mu)
        assert torch.equal(again, rho) and torch.equal(ev2, ev)
