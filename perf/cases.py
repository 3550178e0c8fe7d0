"""Timed cases of the operator-state path, through the public entry points.

Each case is a dict of plain values; ``prepare`` makes what a program holds
before the call (operator handle with its tables, sector, state), ``run`` is
one pass, ``exact`` the same result in plain float64 torch, ``work`` the bytes
and operations no implementation can avoid.

Kinds:
  apply     H|psi> of a molecular operator in a spin sector
  energy    the fused energy of the same, H|psi> stored by the same pass
  step      operator construction from integrals (Jordan-Wigner, grouping,
            sector, factor tables), then the fused energy
  hubbard   fused energy of a lattice operator: few groups, long rows
  krylov    one short-iterative Lanczos step of a lattice operator
  batch     uneven sector jobs, each its own operator, in one launch
  vqe       energy and adjoint gradient of a rotation ansatz on 2^n amplitudes
  full      H|psi> of a spin chain on the full 2^n space
  product   canonical product of two Pauli sums
"""

import math

import numpy as np
import torch

from paper_2606_28952_amd import api

DTYPES = {"c64": torch.complex64, "c128": torch.complex128}
DT = 0.05  # time step of a propagation
VECTORS = 12  # Lanczos vectors of a step


def listed():
    return [
        # smallest call: 12 qubits, 400 configurations; launch latency
        {"name": "apply-12q-c128", "kind": "apply", "n_orb": 6, "na": 3, "nb": 3, "dtype": "c128", "factored": True},
        # an ordinary energy on an operator used once or twice, for which no
        # factor tables are built; open shell
        {"name": "energy-22q-c64-plain", "kind": "energy", "n_orb": 11, "na": 5, "nb": 6, "dtype": "c64",
         "factored": False},
        # ragged double-precision product: odd orbital count, unequal spins
        {"name": "apply-26q-c128", "kind": "apply", "n_orb": 13, "na": 6, "nb": 5, "dtype": "c128", "factored": True},
        # the 28-qubit sector of the benchmark, the largest molecular one
        {"name": "apply-28q-c64", "kind": "apply", "n_orb": 14, "na": 7, "nb": 7, "dtype": "c64", "factored": True},
        # a new operator per step: small, where construction is everything
        {"name": "step-16q-c128", "kind": "step", "n_orb": 8, "na": 4, "nb": 4, "dtype": "c128", "factored": True},
        # the benchmark's step: construction and fused energy at 28 qubits
        {"name": "step-28q-c64", "kind": "step", "n_orb": 14, "na": 7, "nb": 7, "dtype": "c64", "factored": True},
        # 4 x 4 Hubbard at half filling, 1.33 GB of amplitudes: bandwidth
        {"name": "hubbard-32q-c64", "kind": "hubbard", "rows": 4, "cols": 4, "na": 8, "nb": 8, "dtype": "c64"},
        # propagation of a 3 x 4 lattice in double precision
        {"name": "krylov-24q-c128", "kind": "krylov", "rows": 3, "cols": 4, "na": 6, "nb": 6, "dtype": "c128"},
        # sixteen uneven sectors of 10 to 13 orbitals in one launch
        {"name": "batch-16-c64", "kind": "batch", "jobs": 16, "low": 10, "high": 13, "dtype": "c64"},
        # one evaluation of the variational scan: forward and backward
        {"name": "vqe-24q-c128", "kind": "vqe", "n_orb": 12, "rot": 200, "dtype": "c128"},
        # full space: a 22-site transverse-field Ising chain
        {"name": "full-22q-c64", "kind": "full", "sites": 22, "dtype": "c64"},
        # Pauli algebra alone: the square of a 12-qubit Hamiltonian
        {"name": "product-12q", "kind": "product", "n_orb": 6},
    ]


def _comb(n, k):
    return math.comb(n, k) if 0 <= k <= n else 0


def draw(rng):
    kind = rng.choice(["apply", "apply", "energy", "energy", "step", "hubbard", "krylov", "batch", "vqe", "full",
                       "product"])
    dtype = rng.choice(["c64", "c128"])
    if kind in ("apply", "energy", "step"):
        while True:
            n = rng.randint(4, 14)
            na = min(n - 1, max(1, n // 2 + rng.randint(-3, 2)))
            nb = min(n - 1, max(1, n // 2 + rng.randint(-3, 2)))
            # (7, 7) of 14 orbitals is listed in complex64
            if _comb(n, na) * _comb(n, nb) <= (8_000_000 if dtype == "c128" else 11_800_000):
                break
        return {"kind": kind, "n_orb": n, "na": na, "nb": nb, "dtype": dtype,
                "factored": kind == "step" or rng.random() < 0.7}
    if kind in ("hubbard", "krylov"):
        most = 1_000_000 if kind == "krylov" else 90_000_000
        while True:
            rows, cols = rng.choice([(2, 3), (2, 4), (3, 3), (2, 5), (3, 4), (2, 7), (3, 5), (4, 4)])
            n = rows * cols
            na, nb = rng.randint(2, n // 2 + 1), rng.randint(2, n // 2 + 1)
            if _comb(n, na) * _comb(n, nb) <= most:
                return {"kind": kind, "rows": rows, "cols": cols, "na": na, "nb": nb, "dtype": dtype}
    if kind == "batch":
        low = rng.randint(6, 10)
        return {"kind": "batch", "jobs": rng.randint(3, 16), "low": low, "high": low + rng.randint(1, 3),
                "dtype": dtype}
    if kind == "vqe":
        return {"kind": "vqe", "n_orb": rng.randint(4, 11), "rot": round(2 ** rng.uniform(3, 7.6)), "dtype": dtype}
    if kind == "full":
        return {"kind": "full", "sites": rng.randint(6, 22), "dtype": dtype}
    return {"kind": "product", "n_orb": rng.randint(2, 6), "cut": round(rng.uniform(0.02, 0.12), 4)}


# ------------------------------------------------------------------ inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _molecule(n, gen):
    """Real spatial integrals (h, g) with the symmetries of real orbitals:
    h ~ N(0, 1), one N(0, 0.1^2) draw per 8-fold orbit of (pq|rs)."""
    a = torch.randn(n, n, generator=gen, device="cuda", dtype=torch.float64)
    h = torch.triu(a) + torch.triu(a, 1).T
    raw = 0.1 * torch.randn(n, n, n, n, generator=gen, device="cuda", dtype=torch.float64)
    i = torch.arange(n, device="cuda")
    p, q, r, s = torch.meshgrid(i, i, i, i, indexing="ij")
    b1, l1, b2, l2 = torch.maximum(p, q), torch.minimum(p, q), torch.maximum(r, s), torch.minimum(r, s)
    first = b1 * n + l1 >= b2 * n + l2
    return h, raw[torch.where(first, b1, b2), torch.where(first, l1, l2), torch.where(first, b2, b1),
                  torch.where(first, l2, l1)]


def _spin_orbitals(h, g):
    """Blocked spin-orbital (h1, h2): h2[P,Q,R,S] multiplies a+_P a+_Q a_R a_S / 2."""
    n = h.shape[0]
    k = torch.arange(2 * n, device="cuda")
    sp, spin = k % n, k // n
    h1 = h[sp][:, sp] * (spin[:, None] == spin[None, :])
    P, Q, R, S = torch.meshgrid(k, k, k, k, indexing="ij")
    allowed = (spin[P] == spin[S]) & (spin[Q] == spin[R])
    return h1.contiguous(), torch.where(allowed, g[sp[P], sp[S], sp[Q], sp[R]], torch.zeros((), device="cuda",
                                                                                               dtype=torch.float64))


def _lattice(rows, cols, gen):
    """Periodic Hubbard model (t = 1, U near 4) as spatial integrals."""
    n = rows * cols
    h = torch.zeros(n, n, dtype=torch.float64)
    for r in range(rows):
        for c in range(cols):
            for rr, cc in ((r, (c + 1) % cols), ((r + 1) % rows, c)):
                i, j = r * cols + c, rr * cols + cc
                if i != j:
                    h[i, j] = h[j, i] = -1.0
    u = 4.0 + 0.1 * torch.randn((), generator=gen, device="cuda", dtype=torch.float64)
    g = torch.zeros(n, n, n, n, device="cuda", dtype=torch.float64)
    i = torch.arange(n, device="cuda")
    g[i, i, i, i] = u
    return h.cuda(), g


def _state(dim, dtype, gen):
    v = torch.randn(dim, 2, generator=gen, device="cuda", dtype=torch.float64)
    v /= v.square().sum().sqrt()
    return torch.view_as_complex(v).to(DTYPES[dtype])


def _jobs(case):
    """(n_orb, N_alpha, N_beta) of each job of a batch, uneven by design."""
    out = []
    for i in range(case["jobs"]):
        n = case["low"] + i % (case["high"] - case["low"] + 1)
        e = n + (-2, -1, 0, 1)[(i // 4) % 4]
        out.append((n, (e + e % 2) // 2, (e - e % 2) // 2))
    return out


def _ansatz(n, rot):
    """X and Z masks of excitation strings (Y on the lowest qubit, X on the
    others, Z inside each pair): every single, then doubles, cut to ``rot``."""
    o = n // 2
    occ, vir = [*range(o), *range(n, n + o)], [*range(o, n), *range(n + o, 2 * n)]
    ex = [(i, a) for i in occ for a in vir if i // n == a // n]
    both = [(i, j, a, b) for x, i in enumerate(occ) for j in occ[x + 1:] for y, a in enumerate(vir)
            for b in vir[y + 1:] if i // n + j // n == a // n + b // n]
    both = [both[k] for k in np.random.default_rng(7).permutation(len(both))]
    xs, zs = [], []
    for qs in (ex + both)[:rot]:
        qs = sorted(qs)
        z = 1 << qs[0]
        for a, b in zip(qs[0::2], qs[1::2]):
            z |= ((1 << b) - 1) & ~((1 << (a + 1)) - 1)
        xs.append(sum(1 << q for q in qs))
        zs.append(z)
    return np.array(xs, dtype=np.uint64), np.array(zs, dtype=np.uint64)


def _angles(rot, seed):
    return np.random.default_rng(seed).normal(size=rot) * 0.05


def _reference(n):
    return ((1 << (n // 2)) - 1) * ((1 << n) + 1)


def _chain(case, gen):
    """Coupling and field of the Ising chain J sum Z Z + h sum X."""
    v = torch.randn(2, generator=gen, device="cuda", dtype=torch.float64).tolist()
    return 0.25 + 0.05 * v[0], 1.0 + 0.05 * v[1]


def _chain_sum(n, j, h):
    x = [0] * (n - 1) + [1 << i for i in range(n)]
    z = [3 << i for i in range(n - 1)] + [0] * n
    return api.PauliSum.create(n, np.array(x, np.uint64), np.array(z, np.uint64),
                               np.array([j] * (n - 1) + [h] * n, np.complex128)).canonicalize()


# --------------------------------------------------------- prepare and run


def _operator(n, na, nb, h, g, factored):
    """(grouped operator with its tables, sector)."""
    grouped = api.jw_transform(*_spin_orbitals(h, g)).group()
    space = api.Space.sector(n, na, nb)
    if factored:
        grouped.factor(space)
    return grouped, space


def prepare(case, seed):
    gen, kind = _generator(seed), case["kind"]
    if kind in ("apply", "energy", "step"):
        n, na, nb = case["n_orb"], case["na"], case["nb"]
        h, g = _molecule(n, gen)
        psi = _state(_comb(n, na) * _comb(n, nb), case["dtype"], gen)
        s = {"case": case, "psi": psi, "out": torch.empty_like(psi)}
        if kind == "step":
            return {**s, "integrals": _spin_orbitals(h, g)}
        grouped, space = _operator(n, na, nb, h, g, case["factored"])
        return {**s, "grouped": grouped, "space": space}
    if kind in ("hubbard", "krylov"):
        h, g = _lattice(case["rows"], case["cols"], gen)
        n, na, nb = h.shape[0], case["na"], case["nb"]
        grouped, space = _operator(n, na, nb, h, g, True)
        psi = _state(_comb(n, na) * _comb(n, nb), case["dtype"], gen)
        s = {"case": case, "psi": psi, "grouped": grouped, "space": space}
        if kind == "krylov":
            return {**s, "propagator": api.KrylovPropagator(grouped, space, dtype=DTYPES[case["dtype"]], m=VECTORS)}
        return {**s, "out": torch.empty_like(psi)}
    if kind == "batch":
        jobs = []
        for n, na, nb in _jobs(case):
            h, g = _molecule(n, gen)
            psi = _state(_comb(n, na) * _comb(n, nb), case["dtype"], gen)
            jobs.append((*_operator(n, na, nb, h, g, True), psi, torch.empty_like(psi)))
        return {"case": case, "jobs": jobs, "batch": api.Batch(jobs),
                "energies": torch.zeros(3 * len(jobs), dtype=torch.float64, device="cuda")}
    if kind == "vqe":
        n = case["n_orb"]
        grouped = api.jw_transform(*_spin_orbitals(*_molecule(n, gen))).group()
        x, z = _ansatz(n, case["rot"])
        return {"case": case, "theta": _angles(len(x), seed),
                "vqe": api.VQE(grouped, n, x, z, _reference(n), dtype=DTYPES[case["dtype"]])}
    if kind == "full":
        n = case["sites"]
        psi = _state(1 << n, case["dtype"], gen)
        return {"case": case, "psi": psi, "out": torch.empty_like(psi), "space": api.Space.full(n),
                "grouped": _chain_sum(n, *_chain(case, gen)).group()}
    h, g = _molecule(case["n_orb"], gen)
    return {"case": case, "sum": api.jw_transform(*_spin_orbitals(h, g), eps=case.get("cut", 0.0))}


def run(s):
    kind = s["case"]["kind"]
    if kind in ("apply", "full"):
        return {"out": api.apply_pauli_sum(s["grouped"], s["space"], s["psi"], out=s["out"])}
    if kind in ("energy", "hubbard"):
        return {"energy": api.expval(s["grouped"], s["space"], s["psi"], out=s["out"]), "out": s["out"]}
    if kind == "step":
        c = s["case"]
        grouped = api.jw_transform(*s["integrals"]).group()
        space = api.Space.sector(c["n_orb"], c["na"], c["nb"])
        grouped.factor(space)
        return {"energy": api.expval(grouped, space, s["psi"], out=s["out"]), "out": s["out"]}
    if kind == "krylov":
        return {"info": list(s["propagator"].step(s["psi"], DT)), "psi": s["psi"]}
    if kind == "batch":
        return {"energies": s["batch"].run(s["energies"]), "out": [j[3] for j in s["jobs"]]}
    if kind == "vqe":
        energy, grad = s["vqe"].energy_grad(s["theta"])
        return {"energy": energy, "grad": grad}
    x, z, c = s["sum"].mul(s["sum"]).read()
    return {"x": x.view(np.int64), "z": z.view(np.int64), "c": c}


# -------------------------------------------------------- the same in 64 bits


def _strings(n, k):
    """Spin strings of n orbitals with k ones (every string for k = None), ascending."""
    s = torch.arange(1 << n, device="cuda")
    return s if k is None else s[_popcount(s) == k]


def _popcount(v):
    c = torch.zeros_like(v)
    for b in range(32):
        c += (v >> b) & 1
    return c


def _hops(strings, n):
    """a+_p a_q on the strings: {(p, q): (targets, sources, signs)}, and the
    same concatenated as (flat matrix places, signs, p * n + q)."""
    d = len(strings)
    place = torch.full((1 << n,), -1, device="cuda", dtype=torch.int64)
    place[strings] = torch.arange(d, device="cuda")
    hops = {}
    for p in range(n):
        for q in range(n):
            ok = (strings >> q) & 1
            if p != q:
                ok = ok & ~(strings >> p) & 1
            src = torch.nonzero(ok).reshape(-1)
            t = strings[src]
            lo, hi = min(p, q), max(p, q)
            inside = t & (((1 << hi) - 1) & ~((1 << (lo + 1)) - 1))
            dst = place[t ^ ((1 << p) | (1 << q))] if p != q else src
            hops[p, q] = (dst, src, _parity(inside))
    at = torch.cat([t * d + f for t, f, _ in hops.values()])
    sign = torch.cat([s for _, _, s in hops.values()])
    pair = torch.cat([torch.full_like(f, p * n + q) for (p, q), (_, f, _) in hops.items()])
    return hops, (at, sign, pair)


def _one_body(strings, m, flat):
    """Dense matrix of sum_pq m[p, q] a+_p a_q."""
    d = len(strings)
    at, sign, pair = flat
    out = torch.zeros(d * d, device="cuda", dtype=torch.float64)
    return out.index_add_(0, at, m.reshape(-1)[pair] * sign).view(d, d)


def _same_spin(strings, h, g, hops, flat):
    """One-body and same-spin two-body operator of one spin."""
    k = _one_body(strings, h - 0.5 * torch.einsum("prrq->pq", g), flat)
    for (p, q), (t, f, s) in hops.items():
        k.index_add_(0, t, 0.5 * s[:, None] * _one_body(strings, g[p, q].contiguous(), flat)[f])
    return k


def _product(h, g, sa, sb):
    """H as a function of psi[rows = sa, columns = sb], by float64 dense products."""
    n, da, db = h.shape[0], len(sa), len(sb)
    lattice = int(torch.count_nonzero(g)) == n  # only on-site terms
    (ha, fa), (hb, fb) = _hops(sa, n), _hops(sb, n)
    if lattice:
        ka, kb = _one_body(sa, h, fa), _one_body(sb, h, fb)
        cross = g[0, 0, 0, 0] * _popcount(sa[:, None] & sb[None, :]).to(torch.float64)
    else:
        ka, kb = _same_spin(sa, h, g, ha, fa), _same_spin(sb, h, g, hb, fb)

    def apply(psi):
        v = torch.view_as_real(psi.to(torch.complex128)).permute(2, 0, 1).reshape(2, da, db)
        out = torch.stack([ka @ v[0] + v[0] @ kb.T, ka @ v[1] + v[1] @ kb.T])
        if lattice:
            out += cross * v
        else:
            for p in range(n):
                for q in range(p + 1):  # (pq|rs) = (qp|rs)
                    w = _one_body(sb, g[p, q].contiguous(), fb).T.contiguous()
                    w = torch.stack([v[0] @ w, v[1] @ w])
                    for t, f, s in (ha[k] for k in {(p, q), (q, p)}):
                        out.index_add_(1, t, s[None, :, None] * w[:, f])
        return torch.complex(out[0], out[1])

    return apply


def _energy_of(psi, out):
    e = torch.sum(psi.conj() * out)
    return torch.stack([e.real, e.imag, psi.abs().square().sum()])


def _exact_sector(n, na, nb, h, g, psi):
    sa, sb = _strings(n, na), _strings(n, nb)
    psi = psi.to(torch.complex128)
    out = _product(h, g, sa, sb)(psi.view(len(sa), len(sb))).reshape(-1)
    return _energy_of(psi, out), out


def _exact_krylov(case, gen):
    h, g = _lattice(case["rows"], case["cols"], gen)
    n = h.shape[0]
    sa, sb = _strings(n, case["na"]), _strings(n, case["nb"])
    psi = _state(len(sa) * len(sb), case["dtype"], gen).to(torch.complex128).view(len(sa), len(sb))
    product = _product(h, g, sa, sb)
    norm = psi.abs().square().sum().sqrt()
    mean = torch.sum(psi.conj() * product(psi)).real / norm ** 2
    steps = 4
    for _ in range(steps):  # Taylor series of each quarter step
        term = psi
        for k in range(1, 30):
            term = product(term) * (-1j * DT / steps / k)
            psi = psi + term
    return {"info": [float(norm), float(mean), None, None], "psi": psi.reshape(-1)}


def _parity(v):
    for b in (16, 8, 4, 2, 1):
        v = v ^ (v >> b)
    return 1.0 - 2.0 * (v & 1).to(torch.float64)


def _exact_vqe(case, gen, seed):
    n = case["n_orb"]
    h, g = _molecule(n, gen)
    x, z = ([int(v) for v in m] for m in _ansatz(n, case["rot"]))
    theta = _angles(len(x), seed)
    t = torch.arange(1 << (2 * n), device="cuda", dtype=torch.int32)

    def pauli(k, v):  # (P v)[t] = i^|x & z| (-1)^(z . (t ^ x)) v[t ^ x]
        u = t ^ x[k]
        return (1j ** (bin(x[k] & z[k]).count("1") % 4)) * _parity(u & z[k]) * v[u.long()]

    psi = torch.zeros(len(t), device="cuda", dtype=torch.complex128)
    psi[_reference(n)] = 1.0
    for k in range(len(x)):
        psi = math.cos(theta[k]) * psi + 1j * math.sin(theta[k]) * pauli(k, psi)
    s = _strings(n, None)
    lam = _product(h, g, s, s)(psi.view(len(s), len(s))).reshape(-1)  # H is the same for both spins
    energy = float(torch.sum(psi.conj() * lam).real)
    grad = np.zeros(len(x))
    for k in reversed(range(len(x))):
        image = pauli(k, psi)
        grad[k] = -2.0 * float(torch.sum(lam.conj() * image).imag)
        psi = math.cos(theta[k]) * psi - 1j * math.sin(theta[k]) * image
        lam = math.cos(theta[k]) * lam - 1j * math.sin(theta[k]) * pauli(k, lam)
    return {"energy": energy, "grad": grad}


def exact(case, seed):
    gen, kind = _generator(seed), case["kind"]
    if kind in ("apply", "energy", "step"):
        n, na, nb = case["n_orb"], case["na"], case["nb"]
        h, g = _molecule(n, gen)
        energy, out = _exact_sector(n, na, nb, h, g, _state(_comb(n, na) * _comb(n, nb), case["dtype"], gen))
        return {"out": out} if kind == "apply" else {"energy": energy, "out": out}
    if kind == "hubbard":
        h, g = _lattice(case["rows"], case["cols"], gen)
        n, na, nb = h.shape[0], case["na"], case["nb"]
        energy, out = _exact_sector(n, na, nb, h, g, _state(_comb(n, na) * _comb(n, nb), case["dtype"], gen))
        return {"energy": energy, "out": out}
    if kind == "krylov":
        return _exact_krylov(case, gen)
    if kind == "batch":
        res = []
        for n, na, nb in _jobs(case):
            h, g = _molecule(n, gen)
            res.append(_exact_sector(n, na, nb, h, g, _state(_comb(n, na) * _comb(n, nb), case["dtype"], gen)))
        return {"energies": torch.cat([r[0] for r in res]), "out": [r[1] for r in res]}
    if kind == "vqe":
        return _exact_vqe(case, gen, seed)
    if kind == "full":
        n = case["sites"]
        psi = _state(1 << n, case["dtype"], gen).to(torch.complex128)
        j, h = _chain(case, gen)
        t = torch.arange(1 << n, device="cuda", dtype=torch.int32)
        out = sum(_parity(t & (3 << i)) for i in range(n - 1)) * (j * psi)
        for i in range(n):
            out += h * psi[(t ^ (1 << i)).long()]
        return {"out": out}
    return None  # products are correctly rounded and stay bit for bit the same


# ------------------------------------------------------------- least work


def _connected(n, na, nb):
    """Configurations that a two-body operator connects to one target, itself included."""
    sa, sb = na * (n - na), nb * (n - nb)
    da, db = _comb(na, 2) * _comb(n - na, 2), _comb(nb, 2) * _comb(n - nb, 2)
    return 1 + sa + sb + da + db + sa * sb


def _lattice_hops(rows, cols, k):
    """Average hops of k particles on the periodic lattice."""
    n, bonds = rows * cols, set()
    for r in range(rows):
        for c in range(cols):
            for j in (r * cols + (c + 1) % cols, (r + 1) % rows * cols + c):
                if j != r * cols + c:
                    bonds.add(frozenset((r * cols + c, j)))
    return len(bonds) * 2.0 * k * (n - k) / (n * (n - 1))


def work(case):
    kind = case["kind"]
    b = 16 if case.get("dtype") == "c128" else 8
    if kind in ("apply", "energy", "step"):
        n, na, nb = case["n_orb"], case["na"], case["nb"]
        d = _comb(n, na) * _comb(n, nb)
        more = 8 * (2 * n) ** 4 if kind == "step" else 0
        return {"bytes": 2.0 * d * b + more, "flops": 4.0 * d * _connected(n, na, nb)}
    if kind in ("hubbard", "krylov"):
        n = case["rows"] * case["cols"]
        d = _comb(n, case["na"]) * _comb(n, case["nb"])
        f = 4.0 * d * (1 + sum(_lattice_hops(case["rows"], case["cols"], case[k]) for k in ("na", "nb")))
        if kind == "hubbard":
            return {"bytes": 2.0 * d * b, "flops": f}
        return {"bytes": 2.0 * (VECTORS + 1) * d * b, "flops": VECTORS * f + 8.0 * d * VECTORS * (VECTORS + 1)}
    if kind == "batch":
        w = [(_comb(n, na) * _comb(n, nb), _connected(n, na, nb)) for n, na, nb in _jobs(case)]
        return {"bytes": 2.0 * b * sum(d for d, _ in w), "flops": 4.0 * sum(d * c for d, c in w)}
    if kind == "vqe":
        n = case["n_orb"]
        d = 4.0 ** n
        f = sum(4.0 * _comb(n, p) * _comb(n, q) * _connected(n, p, q) for p in range(n + 1) for q in range(n + 1))
        rot = len(_ansatz(n, case["rot"])[0])
        return {"bytes": 4.0 * d * b, "flops": f + rot * d * (3 * 6 + 8)}
    if kind == "full":
        n = case["sites"]
        return {"bytes": 2.0 * b * 2 ** n, "flops": 2.0 ** n * (4 * (n + 1) + n - 1)}
    m = {2: 27, 3: 118, 4: 361, 5: 876, 6: 1819}[case["n_orb"]]
    return {"bytes": 32.0 * m * 3, "flops": 4.0 * m * m}
