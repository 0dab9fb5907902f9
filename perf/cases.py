"""Performance cases of the framework: the calls a tomography program makes, through the
public Python entry points, from a 1-qubit estimate to a 13-qubit one, batches, slabs,
the reduced operator set and the projection onto physical states.

listed() names the cases, draw() gives further ones of the same ranges, prepare() makes
what a program holds before the call, run() is one pass, work() the bytes and operations
the pass cannot do without, exact() the same outputs from plain float64 torch.

A case's fields:
  kind   estimate | noalloc | batch | stream | povm | project
  n      qubits (batch: n_lo .. n_hi over the instances)
  totals uniform (every basis has the same number of shots), given (a total per basis,
         handed to the call) or rows (a total per basis, summed by the call)
  rho    c128 | c64 | none: the precision of the returned matrix, or no matrix
  held   the program keeps output and workspace buffers between calls and checks the
         error flags itself, later; otherwise the call is made with its defaults
         (buffers allocated, flags checked, i.e. the stream synchronised)
"""
import math

import torch

from paper_1602_08604_amd import lre

DEVICE = "cuda"


# ---------------------------------------------------------------------------------
# cases

def listed():
    return [
        # one small register, the plain call of an interactive program: launches and host time
        dict(name="estimate-n4", kind="estimate", n=4, totals="uniform", shots=1000, rho="c128", held=False),
        # a serving loop that must not allocate: the library's own scratch, totals from the rows
        dict(name="noalloc-n7", kind="noalloc", n=7, totals="rows", shots=4000, rho="c128", held=True),
        # eight qubits at 10^4 shots (the small benchmark workload)
        dict(name="estimate-n8", kind="estimate", n=8, totals="uniform", shots=10000, rho="c128", held=True),
        # a mid-size register with lost shots (a total per basis), single-precision matrix
        dict(name="estimate-n10-given-c64", kind="estimate", n=10, totals="given", shots=2000, rho="c64", held=True),
        # the same kind of data one size up, totals left to the call, its default buffers
        dict(name="estimate-n11-rows", kind="estimate", n=11, totals="rows", shots=3000, rho="c128", held=False),
        # twelve qubits at 10^4 shots (the mid benchmark workload)
        dict(name="estimate-n12", kind="estimate", n=12, totals="uniform", shots=10000, rho="c128", held=True),
        # the largest single estimate of which several fit the card: counts 0..12, a total per basis
        dict(name="estimate-n13-given", kind="estimate", n=13, totals="given", shots=0, rho="c128", held=True),
        # 512 independent instances of 3..9 qubits in one tuned launch (the batch benchmark)
        dict(name="batch-512", kind="batch", count=512, n_lo=3, n_hi=9, totals="uniform", rho="c128", tune=True),
        # a handful of runs with per-basis totals, the plan as it comes
        dict(name="batch-40-rows", kind="batch", count=40, n_lo=5, n_hi=9, totals="rows", rho="c128", tune=False),
        # counts arriving slab by slab (the letters of two qubits fixed per slab), already on the device
        dict(name="stream-n12-h2", kind="stream", n=12, h=2, totals="uniform", shots=5000, rho="c128", host=False),
        # a four-outcome measurement per qubit instead of the Pauli bases
        dict(name="povm-n12", kind="povm", n=12, rho="c128", held=True),
        # the physical state closest to an estimate
        dict(name="project-n8", kind="project", n=8, shots=200),
    ]


def _shots(rng):
    return int(round(math.exp(rng.uniform(math.log(100), math.log(10000)))))


def draw(rng):
    kind = rng.choices(["estimate", "noalloc", "batch", "stream", "povm", "project"], [10, 2, 3, 2, 2, 1])[0]
    rho = rng.choices(["c128", "c64", "none"], [6, 2, 2])[0]
    totals = rng.choices(["uniform", "given", "rows"], [5, 2, 2])[0]
    if kind == "estimate":
        n = rng.randint(1, 12)
        return dict(kind=kind, n=n, totals=totals, shots=_shots(rng), rho=rho, held=rng.random() < 0.6)
    if kind == "noalloc":
        return dict(kind=kind, n=rng.randint(1, 10), totals=totals, shots=_shots(rng), rho=rho, held=True)
    if kind == "batch":
        lo = rng.randint(1, 8)
        hi = rng.randint(lo, 9)
        count = int(round(math.exp(rng.uniform(math.log(2), math.log(400)))))
        return dict(kind=kind, count=count, n_lo=lo, n_hi=hi, totals=totals, rho=rho, tune=rng.random() < 0.4)
    if kind == "stream":
        host = rng.random() < 0.3
        n = rng.randint(9, 10 if host else 12)
        return dict(kind=kind, n=n, h=rng.randint(1, min(3, n - 8)), totals=totals, shots=_shots(rng), rho=rho, host=host)
    if kind == "povm":
        return dict(kind=kind, n=rng.randint(1, 13), rho=rho, held=rng.random() < 0.6)
    return dict(kind="project", n=rng.randint(2, 9), shots=rng.choice([100, 200, 500, 1000]))


def _flags(case):
    return {"c128": 0, "c64": lre.LRE_RHO_FP32, "none": lre.LRE_NO_RHO}[case["rho"]]


def _rho_dtype(case):
    return torch.complex64 if case["rho"] == "c64" else torch.complex128


# ---------------------------------------------------------------------------------
# inputs, from the seed alone

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _row_shots(n, totals, shots, gen):
    """Shots of every basis: all equal, or (runs that lost some) 60..100 % of `shots`."""
    if totals == "uniform":
        return torch.full((3 ** n,), shots, dtype=torch.int32, device=DEVICE)
    return torch.randint(max(1, (6 * shots) // 10), shots + 1, (3 ** n,), generator=gen, device=DEVICE, dtype=torch.int32)


def _multinomial(n, row_shots, gen):
    """Measurement counts of a depolarised random product state, int16 [3^n, 2^n]: each
    basis's shots split qubit by qubit with the outcome probabilities of that letter."""
    v = torch.randn(n, 3, generator=gen, device=DEVICE, dtype=torch.float64)
    p_plus = (0.5 + 0.45 * v / v.norm(dim=1, keepdim=True)).float()      # P(+1) per qubit and letter
    out = torch.empty(3 ** n, 2 ** n, dtype=torch.int16, device=DEVICE)
    slab = max(1, (1 << 26) >> n)
    for b0 in range(0, 3 ** n, slab):
        b = torch.arange(b0, min(3 ** n, b0 + slab), device=DEVICE)
        c = row_shots[b].float().unsqueeze(1)
        for k in range(n):
            p = p_plus[k][(b // 3 ** (n - 1 - k)) % 3].unsqueeze(1).expand_as(c).contiguous()
            a = torch.binomial(c, p, generator=gen)
            c = torch.stack((a, c - a), dim=2).flatten(1)
        out[b0:b0 + len(b)] = c.to(torch.int16)
    return out


def _counts(n, totals, shots, seed):
    """(counts int16 [3^n, 2^n], shots argument, totals per basis or None)."""
    gen = _generator(seed)
    if shots == 0:                               # the large workload: i.i.d. counts 0..12
        c = torch.empty(3 ** n, 2 ** n, dtype=torch.int16, device=DEVICE)
        nb = torch.empty(3 ** n, dtype=torch.int32, device=DEVICE)
        for b0 in range(0, 3 ** n, 1 << 17):
            c[b0:b0 + (1 << 17)].random_(0, 13, generator=gen)
            nb[b0:b0 + (1 << 17)] = c[b0:b0 + (1 << 17)].sum(1, dtype=torch.int32)
        return c, 0, nb
    rows = _row_shots(n, totals, shots, gen)
    c = _multinomial(n, rows, gen)
    return c, (shots if totals == "uniform" else 0), (None if totals == "uniform" else rows)


def _instances(case, seed):
    """(n, counts, shots argument, totals) of every instance of a batch: the sizes
    n_lo..n_hi in turn, largest first, shots uniform in 100..10^4."""
    gen = torch.Generator()
    gen.manual_seed(seed)
    ns = [case["n_hi"] - j % (case["n_hi"] - case["n_lo"] + 1) for j in range(case["count"])]
    shots = torch.randint(100, 10001, (case["count"],), generator=gen).tolist()
    return [(n, *_counts(n, case["totals"], s, seed * 1009 + j)) for j, (n, s) in enumerate(zip(ns, shots))]


def _povm(n, seed):
    """Counts 0..59 of all 4^n outcomes, and the tetrahedral measurement's components."""
    c = torch.empty(4 ** n, dtype=torch.int16, device=DEVICE).random_(0, 60, generator=_generator(seed))
    c[0] += 1                                    # never all zero
    t = 1.0 / math.sqrt(3.0)
    bloch = torch.tensor([[t, t, t], [t, -t, -t], [-t, t, -t], [-t, -t, t]], dtype=torch.float64)
    G = 0.5 * torch.cat((torch.ones(4, 1, dtype=torch.float64), bloch), dim=1)
    return c, G.to(DEVICE)


def _as_counts(c):
    return c.view(torch.uint16)


# ---------------------------------------------------------------------------------
# the calls

def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("estimate", "noalloc"):
        n, flags = case["n"], _flags(case)
        c, shots, nb = _counts(n, case["totals"], case["shots"], seed)
        s.update(counts=_as_counts(c), shots=shots, nb=nb if case["totals"] == "given" else None, flags=flags,
                 coef=None, rho=None, ws=None)
        if case["held"]:
            s["coef"] = torch.empty(4 ** n, dtype=torch.float64, device=DEVICE)
            if case["rho"] != "none":
                s["rho"] = torch.empty(2 ** n, 2 ** n, dtype=_rho_dtype(case), device=DEVICE)
            if kind == "estimate":
                s["ws"] = torch.empty(max(1, lre.workspace_bytes(n, shots, flags)), dtype=torch.uint8, device=DEVICE)
    elif kind == "batch":
        inst = _instances(case, seed)
        flags = _flags(case)
        sizes = [4 ** i[0] for i in inst]
        s["coef"] = torch.zeros(sum(sizes), dtype=torch.float64, device=DEVICE)
        coefs = list(s["coef"].split(sizes))
        rhos = None
        s["rho"] = None
        if case["rho"] != "none":
            # 4^n complex numbers per instance, each matrix at a 16-byte boundary (4^n is even)
            s["rho"] = torch.zeros(sum(sizes), dtype=_rho_dtype(case), device=DEVICE)
            rhos = [r.view(2 ** i[0], 2 ** i[0]) for r, i in zip(s["rho"].split(sizes), inst)]
        s["plan"] = lre.Batch([_as_counts(i[1]) for i in inst], [i[2] for i in inst], flags=flags, coefs=coefs, rhos=rhos,
                              n_per_basis=[i[3] if case["totals"] == "given" else None for i in inst])
        s["plan"].workspace()
        if case["tune"]:
            s["plan"].tune(reps=2)
    elif kind == "stream":
        n, h = case["n"], case["h"]
        c, shots, nb = _counts(n, case["totals"], case["shots"], seed)
        flags = _flags(case) | (lre.LRE_STREAM_HOST if case["host"] else 0)
        s["stream"] = lre.Stream(n, h, shots, flags=flags)
        s["stream"].workspace()
        if case["totals"] != "given":
            nb = None
        if case["host"]:
            c = torch.empty(c.shape, dtype=c.dtype, pin_memory=True).copy_(c)
            nb = None if nb is None else torch.empty(nb.shape, dtype=nb.dtype, pin_memory=True).copy_(nb)
        rows = 3 ** (n - h)
        s["slabs"] = list(_as_counts(c).split(rows))
        s["nbs"] = [None] * len(s["slabs"]) if nb is None else list(nb.split(rows))
        s["coef"] = torch.empty(4 ** n, dtype=torch.float64, device=DEVICE)
        s["rho"] = None if case["rho"] == "none" else torch.empty(2 ** n, 2 ** n, dtype=_rho_dtype(case), device=DEVICE)
    elif kind == "povm":
        n, flags = case["n"], _flags(case)
        c, G = _povm(n, seed)
        s.update(counts=_as_counts(c), G=G, flags=flags, coef=None, rho=None, ws=None)
        if case["held"]:
            s["coef"] = torch.empty(4 ** n, dtype=torch.float64, device=DEVICE)
            if case["rho"] != "none":
                s["rho"] = torch.empty(2 ** n, 2 ** n, dtype=_rho_dtype(case), device=DEVICE)
            need = int(lre.lib().lre_povm_workspace_bytes(n, flags))
            s["ws"] = torch.empty(max(1, need), dtype=torch.uint8, device=DEVICE)
    else:
        n = case["n"]
        c, _, nb = _counts(n, "uniform", case["shots"], seed)
        s["mu"] = _ref_rho(_ref_coef(c, n, case["shots"], nb), n)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "estimate":
        return lre.estimate(s["counts"], s["shots"], n_per_basis=s["nb"], flags=s["flags"], coef=s["coef"], rho=s["rho"],
                            workspace=s["ws"], check=not case["held"])
    if kind == "noalloc":
        return lre.estimate_noalloc(s["counts"], s["shots"], s["coef"], s["rho"], n_per_basis=s["nb"], flags=s["flags"],
                                    check=False)
    if kind == "batch":
        s["plan"].run()
        return s["coef"], s["rho"]
    if kind == "stream":
        st = s["stream"]
        st.begin(s["coef"])
        push = st.push_host if case["host"] else st.push
        for k, (slab, nb) in enumerate(zip(s["slabs"], s["nbs"])):
            push(k, slab, nb)
        return st.finish(s["rho"], check=False)
    if kind == "povm":
        return lre.povm_estimate(s["counts"], s["G"], flags=s["flags"], coef=s["coef"], rho=s["rho"], workspace=s["ws"],
                                 check=not case["held"])
    return lre.project(s["mu"])


# ---------------------------------------------------------------------------------
# what a pass cannot do without

def _rho_bytes(case, n):
    return {"c128": 16, "c64": 8, "none": 0}[case["rho"]] * 4 ** n


def _estimate_work(case, n):
    b = 2 * 6 ** n + 8 * 4 ** n + _rho_bytes(case, n) + (4 * 3 ** n if case["totals"] == "given" else 0)
    # folding a qubit: 8 additions for each 6 values that become 4; the matrix: a
    # transform of n additions per entry and its last combination
    f = sum(8 * 6 ** (n - k) * 4 ** (k - 1) for k in range(1, n + 1)) + 4 ** n
    if case["rho"] != "none":
        f += (n + 4) * 4 ** n
    return b, f


def work(case):
    kind = case["kind"]
    if kind in ("estimate", "noalloc", "stream"):
        b, f = _estimate_work(case, case["n"])
    elif kind == "batch":
        per = [_estimate_work(case, case["n_hi"] - j % (case["n_hi"] - case["n_lo"] + 1)) for j in range(case["count"])]
        b, f = (sum(p[i] for p in per) for i in (0, 1))
    elif kind == "povm":
        n = case["n"]
        b = (2 + 8) * 4 ** n + _rho_bytes(case, n)
        f = 7 * n * 4 ** n + ((n + 4) * 4 ** n if case["rho"] != "none" else 0)
    else:
        d = 2 ** case["n"]
        b = 2 * 16 * d * d + 8 * d
        f = 8 * d ** 3 * (2 / 3 + 1 + 0.5)       # tridiagonal form, eigenvectors, half of them reassembled
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------------
# the same outputs in float64 with plain torch

def _fold_lowest(t, h, l):
    """[3^h, 2^h, 4^l] -> [3^(h-1), 2^(h-1), 4^(l+1)]: the lowest raw qubit folded."""
    t = t.reshape(3 ** (h - 1), 3, 2 ** (h - 1), 2, 4 ** l)
    even = (t[:, :, :, 0] + t[:, :, :, 1]).sum(1)                        # letter I
    odd = (t[:, :, :, 0] - t[:, :, :, 1]).transpose(1, 2)                # letters X, Y, Z
    return torch.cat((even.unsqueeze(2), odd), dim=2).reshape(3 ** (h - 1), 2 ** (h - 1), 4 ** (l + 1))


def _ref_coef(c, n, shots, nb):
    """Pauli coefficients of counts int16 [3^n, 2^n] (every count below 2^15)."""
    top = min(n - 1, max(0, n - 10))             # the letters and outcomes of the top qubits, piece by piece
    np_ = n - top
    pieces = torch.empty(3 ** top, 2 ** top, 4 ** np_, dtype=torch.float64, device=c.device)
    for b in range(3 ** top):
        rows = slice(b * 3 ** np_, (b + 1) * 3 ** np_)
        for o in range(2 ** top):
            t = c[rows, o * 2 ** np_:(o + 1) * 2 ** np_].double()
            if nb is not None:
                t = t / nb[rows].double().unsqueeze(1)
            for k in range(np_):
                t = _fold_lowest(t, np_ - k, k)
            pieces[b, o] = t.reshape(-1)
    t = pieces
    for k in range(top):
        t = _fold_lowest(t, top - k, np_ + k)
    div = torch.ones(1, dtype=torch.float64, device=c.device)
    one = torch.tensor([3.0, 1.0, 1.0, 1.0], dtype=torch.float64, device=c.device)
    for _ in range(n):
        div = (div.unsqueeze(1) * one).reshape(-1)
    return t.reshape(-1) / (div if nb is not None else div * shots)


def _ref_rho(coef, n):
    """The matrix 2^-n sum_a e_a sigma_a, complex128 [2^n, 2^n]."""
    t = coef.to(torch.complex128).reshape(1, 1, -1)
    for k in range(n):
        r, m = 2 ** k, 4 ** (n - k - 1)
        v = t.reshape(r, r, 4, m)
        new = torch.empty(r, 2, r, 2, m, dtype=t.dtype, device=t.device)
        new[:, 0, :, 0] = v[:, :, 0] + v[:, :, 3]
        new[:, 1, :, 1] = v[:, :, 0] - v[:, :, 3]
        new[:, 0, :, 1] = v[:, :, 1] - 1j * v[:, :, 2]
        new[:, 1, :, 0] = v[:, :, 1] + 1j * v[:, :, 2]
        t = new.reshape(2 * r, 2 * r, m)
    return t.reshape(2 ** n, 2 ** n) / 2 ** n


def exact(case, seed):
    kind = case["kind"]
    if kind in ("estimate", "noalloc", "stream"):
        n = case["n"]
        c, shots, nb = _counts(n, case["totals"], case["shots"], seed)
        coef = _ref_coef(c, n, shots, nb)
        return coef, (None if case["rho"] == "none" else _ref_rho(coef, n))
    if kind == "batch":
        coefs, rhos = [], []
        for n, c, shots, nb in _instances(case, seed):
            coefs.append(_ref_coef(c, n, shots, nb))
            if case["rho"] != "none":
                rhos.append(_ref_rho(coefs[-1], n).reshape(-1))
        return torch.cat(coefs), (torch.cat(rhos) if rhos else None)
    if kind == "povm":
        n = case["n"]
        c, G = _povm(n, seed)
        M = 2.0 * torch.linalg.solve(G.cpu().T @ G.cpu(), G.cpu().T).to(DEVICE)
        t = c.double()
        for k in range(n):
            v = t.reshape(4 ** (n - 1 - k), 4, 4 ** k)
            t = sum(M[:, j].reshape(1, 4, 1) * v[:, j:j + 1] for j in range(4)).reshape(-1)
        coef = t / c.sum(dtype=torch.int64).double()
        return coef, (None if case["rho"] == "none" else _ref_rho(coef, n))
    mu = prepare(case, seed)["mu"].cpu()
    w, V = torch.linalg.eigh(mu)
    a, k = 0.0, len(w)
    lam = w.clone()
    for i in range(len(w)):
        if float(w[i]) + a / k >= 0.0:
            lam[i:] = w[i:] + a / k
            break
        a += float(w[i])
        k -= 1
        lam[i] = 0.0
    return ((V * lam) @ V.conj().T).to(DEVICE), w.to(DEVICE)
