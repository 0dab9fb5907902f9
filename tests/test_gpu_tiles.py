"""The counts pass in sub-tiles and the pass that ends a small plan (5 or more qubits), at
the sizes where their plans change: one workgroup (n <= 5), single sub-tiles (6 to 8
qubits), 6-qubit tiles (9), 7-qubit tiles in blocks that cover part of a row group (10), one
that straddle row groups (11, 12), with each of the accumulator types.

Uniform shots: exact integer numerators, compared with eq. (3)'s sums evaluated in int64 by
NumPy mode products (equality).  Per-basis totals: every coefficient is a sum of at most 3^n
terms S_b / N_b of magnitude <= 1, divided by 3^(n-w); a binary64 sum of M such terms by any
tree is off by at most (depth) 2^-53 of their mean magnitude, depth < 8 n additions and two
roundings for the reciprocal and the product, so 16 n 2^-53 < 3e-14 bounds the difference of
two orders; the bar is 1e-13."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1602_08604_amd import lre as L  # noqa: E402

DEV = "cuda:0"
TOL = 1e-13


def fold(x, n):
    """Mode products of eq. (3) on [3^n, 2^n] (int64 or float64), qubit by qubit from the
    lowest: [B, S, A] -> [B / 3, S / 2, 4 A]."""
    t = x.reshape(3 ** n, 2 ** n, 1)
    for k in range(n):
        b, s, a = 3 ** (n - 1 - k), 2 ** (n - 1 - k), 4 ** k
        t = t.reshape(b, 3, s, 2, a)
        even = (t[:, :, :, 0] + t[:, :, :, 1]).sum(1)
        odd = (t[:, :, :, 0] - t[:, :, :, 1]).transpose(1, 2)
        t = torch.cat((even.unsqueeze(2), odd), 2).reshape(b, s, 4 * a)
    return t.reshape(-1)


def divisor(n):
    d = torch.ones(1, dtype=torch.float64, device=DEV)
    for _ in range(n):
        d = (d.unsqueeze(1) * torch.tensor([3.0, 1.0, 1.0, 1.0], dtype=torch.float64, device=DEV)).reshape(-1)
    return d


def uniform_counts(n, hi, seed):
    """Rows that are rotations of one random row of counts 0..hi: one total for all."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    row = torch.randint(0, hi + 1, (2 ** n,), generator=g, device=DEV)
    off = torch.randint(0, 2 ** n, (3 ** n, 1), generator=g, device=DEV)
    idx = (torch.arange(2 ** n, device=DEV) + off) % 2 ** n
    return row[idx], int(row.sum())


def as_uint16(c):
    return c.to(torch.int32).to(torch.uint16)


@pytest.mark.parametrize("n,hi", [(1, 9), (2, 9), (3, 9), (4, 9), (5, 9), (5, 65535), (6, 9), (7, 30), (8, 9), (8, 65535),
                                  (9, 12), (9, 65535), (10, 3), (10, 65535), (11, 2), (11, 65535)])
def test_numerators_exact(n, hi):
    print(f"[tiles uniform n={n} counts <= {hi}]", flush=True)
    c, shots = uniform_counts(n, hi, 100 * n + hi % 97)
    T = L.pauli_sums(as_uint16(c), shots)
    want = fold(c, n)
    assert torch.equal(T, want)
    coef, _ = L.estimate(as_uint16(c), shots, flags=L.LRE_NO_RHO)
    assert torch.equal(coef, want.double() / (divisor(n) * shots))


@pytest.mark.parametrize("given", [True, False])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11])
def test_per_basis(n, given):
    print(f"[tiles per-basis n={n} given={given}]", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    c = torch.randint(0, 40, (3 ** n, 2 ** n), generator=g, device=DEV)
    c[:, 0] += 1
    nb = c.sum(1)
    want = fold(c.double() / nb.double().unsqueeze(1), n) / divisor(n)
    coef, _ = L.estimate(as_uint16(c), 0, n_per_basis=nb.to(torch.int32) if given else None, flags=L.LRE_NO_RHO)
    assert (coef - want).abs().max().item() <= TOL


@pytest.mark.parametrize("n", [2, 5, 6, 8, 9, 10, 11, 12])
def test_every_row_is_checked(n):
    """A wrong total in the first, a middle and the last row is reported, for uniform shots
    and for given totals; an empty row too."""
    print(f"[tiles row check n={n}]", flush=True)
    c = as_uint16(torch.ones(3 ** n, 2 ** n, dtype=torch.int32, device=DEV))
    nb = torch.full((3 ** n,), 2 ** n, dtype=torch.int32, device=DEV)
    L.estimate(c, 2 ** n, flags=L.LRE_NO_RHO)
    L.estimate(c, 0, n_per_basis=nb, flags=L.LRE_NO_RHO)
    v = c.view(torch.int16)
    for b in (0, 3 ** n // 2, 3 ** n - 1):
        v[b, 2 ** n - 1] += 1
        for kw in ({"shots": 2 ** n}, {"shots": 0, "n_per_basis": nb}):
            with pytest.raises(L.LreError) as e:
                L.estimate(c, flags=L.LRE_NO_RHO, **kw)
            assert e.value.status == L.LRE_E_SHOTS
        v[b] = 0
        with pytest.raises(L.LreError) as e:
            L.estimate(c, 0, flags=L.LRE_NO_RHO)
        assert e.value.status == L.LRE_E_EMPTY_BASIS
        v[b] = 1
    L.estimate(c, 2 ** n, flags=L.LRE_NO_RHO)


@pytest.mark.parametrize("n,h,shots", [(9, 1, 0), (10, 1, 30), (10, 2, 0), (11, 1, 20), (11, 3, 0), (12, 2, 15)])
def test_stream_segments_together(n, h, shots):
    """A slab's segments run in shared launches: the same sums as the whole instance."""
    print(f"[tiles stream n={n} h={h}]", flush=True)
    c, total = uniform_counts(n, 2, 7 * n + h)
    c = as_uint16(c)
    shots = total if shots else 0
    s = L.Stream(n, h, shots, flags=L.LRE_NO_RHO)
    s.begin()
    rows = 3 ** (n - h)
    for k in reversed(range(3 ** h)):
        s.push(k, c[k * rows:(k + 1) * rows])
    coef, _ = s.finish()
    want, _ = L.estimate(c, shots, flags=L.LRE_NO_RHO)
    if shots:
        assert torch.equal(coef, want)
    else:
        assert (coef - want).abs().max().item() <= TOL


@pytest.mark.parametrize("ns,per_basis", [([9], False), ([9, 8, 7, 6, 5], True), ([9] * 14, False), ([9] * 14 + [7, 6, 6, 1], True),
                                          ([6], False), ([6, 6], True), ([2, 4], True), ([8] * 3, False)])
def test_batch_forms(ns, per_basis):
    """A new plan (one launch per stage) against the single instances: 6-qubit tiles with up
    to 3 qubits left (few instances), 7-qubit tiles (14 of 9 qubits), instances of one tile,
    none at all; per-basis totals, given and from the rows, beside uniform shots."""
    print(f"[tiles batch {ns} per-basis={per_basis}]", flush=True)
    counts, shots, nbs = [], [], []
    for j, n in enumerate(ns):
        c, total = uniform_counts(n, 3, 31 * j + n)
        pb = per_basis and j % 3 != 1
        if pb:
            c[:, 0] += 1 + torch.arange(3 ** n, device=DEV) % 5
        counts.append(as_uint16(c))
        shots.append(0 if pb else total)
        nbs.append(c.sum(1).to(torch.int32) if pb and j % 2 else None)
    b = L.Batch(counts, shots, n_per_basis=nbs)
    assert b.tiles["staged"] == 1
    for tiles_per_block in (16, 1, 3):
        b.set_tiles(1, tiles_per_block, 432, 1, 0, 1)
        for c, r in zip(b.coefs, b.rhos):
            c.fill_(7.0)
            r.fill_(7.0)
        b.run(check=True)
        for j in range(len(ns)):
            coef, rho = L.estimate(counts[j], shots[j], n_per_basis=nbs[j])
            if shots[j]:
                assert torch.equal(b.coefs[j], coef) and torch.equal(b.rhos[j], rho)
            else:
                assert (b.coefs[j] - coef).abs().max().item() <= TOL
                assert (b.rhos[j] - rho).abs().max().item() <= TOL
    # a wrong total is reported, in the first and the last instance
    for j in (0, len(ns) - 1):
        v = counts[j].view(torch.int16)
        v[3 ** ns[j] // 2] += 1
        if shots[j] or nbs[j] is not None:
            b.run()
            with pytest.raises(L.LreError) as e:
                L.check_flags(DEV)
            assert e.value.status == L.LRE_E_SHOTS
        v[3 ** ns[j] // 2] -= 1
    b.run(check=True)
    b.close()


@pytest.mark.parametrize("n", [5, 6, 7, 8, 9])
def test_empty_row_is_reported(n):
    """Totals formed from the rows: an empty row anywhere (the first, one in the middle, the
    last) is reported, a row with a single count is not."""
    for row in (0, 3 ** n // 2, 3 ** n - 1):
        print(f"[tiles empty row n={n} row={row}]", flush=True)
        c = torch.ones((3 ** n, 2 ** n), dtype=torch.int64, device=DEV)
        c[row] = 0
        with pytest.raises(L.LreError) as e:
            L.estimate(as_uint16(c), 0, flags=L.LRE_NO_RHO)
        assert e.value.status == L.LRE_E_EMPTY_BASIS
        c[row, -1] = 1
        coef, _ = L.estimate(as_uint16(c), 0, flags=L.LRE_NO_RHO)
        assert abs(coef[0].item() - 1.0) <= TOL
