"""The work that programs have this library do, as cases that can be timed and checked.

Inputs are synthetic: random integrals, and block operators with the operator list, sector changes and
sector sizes of a DMRG bond and random values. `exact` computes what a pass returns in 64 bits from
the definitions, with dense torch matrices over all sectors.
"""
import math
import random

import numpy as np
import torch

import paper_2001_04890_amd as dm

DEV = "cuda:0"
N_FACTORS = 16


# ---------------------------------------------------------------------------------------- the cases
def listed():
    return [
        # A bond near the end of the lattice or of an early sweep: a few hundred tasks of a few states,
        # where launches and latency are all there is.
        _hpsi("hpsi_f64_small", 10, 5, 5, 30, 1.5, 0.3),
        # An ordinary active space, odd sizes, unequal spins.
        _hpsi("hpsi_f64_mid", 17, 9, 7, 333, 1.4, 0.4),
        # The middle bond of 24 orbitals at bond dimension 1024, uneven sectors as sweeps leave them: the
        # matvec that a production solve repeats hundreds of times.
        _hpsi("hpsi_f64_large", 24, 12, 12, 1024, 1.35, 0.3),
        # One device's share of the operator pairs of a 76-orbital problem at bond dimension 6000:
        # sectors of some 400 states.
        _hpsi("hpsi_f64_share", 76, 57, 56, 6000, 1.5, 0.0, pairs=20),
        # The large bond in split precision, as Davidson's first iterations run it.
        _hpsi("hpsi_split_large", 24, 12, 12, 1024, 1.35, 0.3, split=True),
        # Independent problems merged into one handle and launched as one graph.
        {"name": "hpsi_batch", "kind": "batch", "n": 12, "L0": 10, "L1": 18, "M0": 40, "M1": 300, "split": False},
        # A whole solve as the early sweeps cap it: 16 iterations from a random start vector.
        {"name": "davidson_mid", "kind": "davidson", "L": 16, "na": 8, "nb": 8, "M": 200, "sigma": 1.4, "uneven": 0.4,
         "iters": 16},
        # The truncation's density matrix at the large bond.
        {"name": "rdm_large", "kind": "rdm", "L": 24, "na": 12, "nb": 12, "M": 1024, "sigma": 1.5, "uneven": 0.2,
         "side": 0},
        # Operators of the enlarged block (4 M states) taken into the kept basis of M states.
        {"name": "renorm_blocks_large", "kind": "renorm", "L": 24, "na": 12, "nb": 12, "M": 1024, "sigma": 1.5,
         "uneven": 0.2, "ops": 12},
        # A block grown by one site and renormalized, from host blocks to a host block.
        {"name": "grow_mid", "kind": "grow", "L": 14, "na": 7, "nb": 7, "M": 150, "sigma": 1.4, "uneven": 0.3, "side": 0},
        # One application of the learned preconditioner's network to every coefficient of a large psi.
        {"name": "mlp_forward", "kind": "mlp_forward", "rows": 660770},
        # One training minibatch of that network: loss and gradient.
        {"name": "mlp_grad", "kind": "mlp_grad", "rows": 4096},
    ]


def _hpsi(name, L, na, nb, M, sigma, uneven, pairs=0, split=False):
    return {"name": name, "kind": "hpsi", "L": L, "na": na, "nb": nb, "M": M, "sigma": sigma, "uneven": uneven,
            "pairs": pairs, "split": split, "graph": False}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _bond_of(rng, L0, L1, M0, M1):
    L = rng.randint(L0, L1)
    return {"L": L, "na": L // 2 + rng.randint(-1, 1), "nb": L // 2 + rng.randint(-1, 1), "M": _log_int(rng, M0, M1),
            "sigma": round(rng.uniform(1.2, 1.7), 2), "uneven": round(rng.uniform(0.0, 0.5), 2)}


def draw(rng):
    kind = rng.choice(["hpsi"] * 4 + ["share", "batch", "davidson", "rdm", "renorm", "grow", "mlp_forward", "mlp_grad"])
    if kind == "hpsi":
        return {"kind": kind, **_bond_of(rng, 8, 24, 16, 1024), "pairs": 0, "split": rng.random() < 0.3,
                "graph": rng.random() < 0.3}
    if kind == "share":
        M = _log_int(rng, 1500, 5000)
        return {"kind": "hpsi", "L": 76, "na": 57, "nb": 56, "M": M, "sigma": 1.5, "uneven": round(rng.uniform(0.0, 0.2), 2),
                "pairs": rng.randint(4, 20), "split": rng.random() < 0.3, "graph": False}
    if kind == "batch":
        L0 = rng.randint(8, 14)
        return {"kind": kind, "n": rng.randint(3, 12), "L0": L0, "L1": L0 + rng.randint(0, 4), "M0": rng.randint(20, 60),
                "M1": _log_int(rng, 80, 300), "split": rng.random() < 0.3}
    if kind == "davidson":
        return {"kind": kind, **_bond_of(rng, 8, 18, 30, 300), "iters": rng.randint(8, 30)}
    if kind == "rdm":
        return {"kind": kind, **_bond_of(rng, 10, 26, 30, 1100), "side": rng.randint(0, 1)}
    if kind == "renorm":
        return {"kind": kind, **_bond_of(rng, 10, 26, 30, 1100), "ops": rng.randint(1, 12)}
    if kind == "grow":
        return {"kind": kind, **_bond_of(rng, 8, 14, 20, 150), "side": rng.randint(0, 1)}
    return {"kind": kind, "rows": _log_int(rng, 700, 600000) if kind == "mlp_forward" else _log_int(rng, 300, 8192)}


# ---------------------------------------------------------------------------------- a bond's structure
def _sectors(k, na, nb, L, M, sigma, uneven, tag):
    """(quantum numbers, dimensions) of a block of k orbitals holding about M states: Gaussian weights about
    the filling, times log-normal factors that make them as uneven as sweeps do, within the number of
    determinants of each sector."""
    r = np.random.RandomState(1000 * L + 7 * M + tag)
    qn = [(p, q) for p in range(k + 1) for q in range(k + 1)]
    w = np.array([math.exp(-((p - na * k / L) ** 2 + (q - nb * k / L) ** 2) / (2 * sigma ** 2)) for p, q in qn])
    w *= np.exp(uneven * r.standard_normal(len(qn)))
    cap = np.array([min(math.comb(k, p) * math.comb(k, q), M) for p, q in qn], dtype=np.int64)
    dims = np.zeros(len(qn), dtype=np.int64)
    for _ in range(40):
        left = min(M, int(cap.sum())) - int(dims.sum())
        if left <= 0:
            break
        ws = w * (dims < cap)
        dims = np.minimum(cap, dims + np.maximum(0, np.rint(left * ws / ws.sum())).astype(np.int64))
    keep = dims > 0
    if not keep.any():
        keep[int(np.argmax(w))] = True
        dims = np.maximum(dims, keep)
    return [q for q, s in zip(qn, keep) if s], [int(d) for d, s in zip(dims, keep) if s]


def _delta(kind, i, j):
    d = [0, 0]
    for idx, sign in {"H": (), "C": ((i, 1),), "S": ((i, 1),), "U": ((i, -1),), "A": ((i, 1), (j, 1)), "P": ((i, -1), (j, -1)),
                      "B": ((i, 1), (j, -1)), "Q": ((j, 1), (i, -1))}[kind]:
        d[idx % 2] += sign
    return tuple(d)


class _Op:
    def __init__(self, kind, i, j, rows):
        self.kind, self.i0, self.i1, self.rows = kind, i, j, rows


class _Block:
    """One block's operators as the library takes them: a flat host array and a table per operator."""

    def __init__(self, side, L, site, na, nb, M, sigma, uneven, pairs=0, only=None):
        self.right = side == "right"
        k = L - site - 2 if self.right else site
        self.sec, self.dims = _sectors(k, na, nb, L, M, sigma, uneven, int(self.right)) if k else ([(0, 0)], [1])
        self.index = {q: s for s, q in enumerate(self.sec)}
        self.qn, self.dim = np.array(self.sec, dtype=np.int32), np.array(self.dims, dtype=np.int32)
        self.n_sec = len(self.sec)
        self.start = np.concatenate([[0], np.cumsum(self.dims)]).astype(int)
        keys, mine = [("H", -1, -1)], range(2 * (site + 2), 2 * L) if self.right else range(2 * site)
        out, n = range(2 * (site + 2)), pairs or None
        pair = out if self.right and not pairs else range(2 * site)
        lower = [(p, q) for p in pair for q in pair if p < q][:n] if self.right or pairs else [(p, q) for p in mine for q in mine if p < q]
        upper = [(p, q) for p in pair for q in pair if p <= q][:n] if self.right or pairs else [(p, q) for p in mine for q in mine if p <= q]
        if not pairs:
            keys += [("C", p, -1) for p in mine]
            keys += [("U", p, -1) for p in out] if self.right else [("S", p, -1) for p in range(2 * site, 2 * L)]
        keys += [("P" if self.right else "A", p, q) for p, q in lower] + [("Q" if self.right else "B", p, q) for p, q in upper]
        if only:
            keys = [key for key in keys if key[0] in only]
        self.ops, off = [], 0
        for key in keys:
            d, rows = _delta(*key), []
            for si, q in enumerate(self.sec):
                so = self.index.get((q[0] + d[0], q[1] + d[1]))
                if so is not None:
                    rows.append((so, si, off))
                    off += self.dims[so] * self.dims[si]
            self.ops.append(_Op(*key, rows))
        self.size, self.at = off, {(o.kind, o.i0, o.i1): o for o in self.ops}
        self.data = None

    def fill(self, seed):
        """Values: block Hamiltonians a rising diagonal with small symmetric noise, the others normal with
        variance 0.04 / (number of columns), so that sums over states keep one size."""
        g = torch.Generator(device=DEV).manual_seed(seed)
        rows = [r for o in self.ops for r in o.rows]
        count = torch.tensor([self.dims[so] * self.dims[si] for so, si, _ in rows] or [0], device=DEV)
        scale = torch.tensor([0.2 / math.sqrt(self.dims[si]) for _, si, _ in rows] or [0.0], device=DEV, dtype=torch.float64)
        v = torch.randn(self.size, device=DEV, dtype=torch.float64, generator=g)
        v *= torch.repeat_interleave(scale, count)
        self.data = v.cpu().numpy()
        r = np.random.RandomState(seed % (1 << 31))
        for o in self.ops:
            if o.kind == "H" or (o.kind in "BQ" and o.i0 == o.i1):
                for so, si, off in o.rows:
                    m = self.data[off:off + self.dims[si] ** 2].reshape(self.dims[si], -1)
                    m[:] = 0.5 * (m + m.T)
                    if o.kind == "H":
                        m *= 0.25
                        m[np.diag_indices_from(m)] += np.sort(r.uniform(0, 6, size=self.dims[si]))
        return self

    def flatten(self):
        return self.data, [o.rows for o in self.ops]

    def dense(self):
        """{operator: its matrix over all states of the block}"""
        v, got = torch.from_numpy(self.data).to(DEV), {}
        for key, o in self.at.items():
            m = torch.zeros(self.start[-1], self.start[-1], dtype=torch.float64, device=DEV)
            for so, si, off in o.rows:
                r, c = self.dims[so], self.dims[si]
                m[self.start[so]:self.start[so + 1], self.start[si]:self.start[si + 1]] = v[off:off + r * c].view(r, c)
            got[key] = m
        return got

    def parity(self):
        return torch.tensor([1.0 - 2.0 * ((p + q) % 2) for (p, q), d in zip(self.sec, self.dims) for _ in range(d)],
                            dtype=torch.float64, device=DEV)


def _integrals(L, seed):
    r = np.random.RandomState(seed % (1 << 31))
    sym = lambda a: np.triu(a) + np.triu(a, 1).swapaxes(-1, -2)  # noqa: E731
    h = sym(r.standard_normal((L, L))) - np.diag(2.0 * np.arange(L) / L)
    b = sym(0.3 * r.standard_normal((N_FACTORS, L, L))).reshape(N_FACTORS, L * L)
    return h, (b.T @ b).reshape(L, L, L, L)


def _blocks(case, only=None):
    site = case["L"] // 2 - 1
    return site, [_Block(s, case["L"], site, case["na"], case["nb"], case["M"], case["sigma"], case["uneven"],
                         case.get("pairs", 0), only) for s in ("left", "right")]


SITE_QN = [(0, 0), (1, 0), (0, 1), (1, 1)]


def _layout(case, left, right):
    """(a, b, c, d) of psi's blocks in their order: those whose electrons add up."""
    got = []
    for a, qa in enumerate(left.sec):
        for b, qb in enumerate(SITE_QN):
            for c, qc in enumerate(SITE_QN):
                d = right.index.get((case["na"] - qa[0] - qb[0] - qc[0], case["nb"] - qa[1] - qb[1] - qc[1]))
                if d is not None:
                    got.append((a, b, c, d))
    return got


# ------------------------------------------------------------------ the Hamiltonian's terms at a bond
def _fermions():
    """Creation operators of the two sites' four spin-orbitals as 16 x 16 matrices, states ordered (b, c)."""
    up, down, one = np.zeros((4, 4)), np.zeros((4, 4)), np.eye(4)
    up[1, 0] = up[3, 2] = 1.0
    down[2, 0], down[3, 1] = 1.0, -1.0
    par = np.diag([1.0, -1.0, -1.0, 1.0])
    return [np.kron(up, one), np.kron(down, one), np.kron(par, up), np.kron(par, down)], np.kron(par, par)


def _terms(L, site, h, eri, left_ops, right_ops):
    """H as a list of (left, site matrix, right, both): left and right are lists of (factor, operator,
    transposed) to be summed, None for the identity; `both`: the transposed term belongs to H too. Sums
    over left or right spin-orbitals with a common rest are taken on the left. Products stand in the
    order left, sites, right; a term whose operators are not there is left out."""
    X, E0, Y = range(2 * site), 2 * site, range(2 * site + 4, 2 * L)
    M = range(E0, E0 + 4)
    cd, _ = _fermions()
    cr = lambda m: cd[m - E0]  # noqa: E731
    an = lambda m: cd[m - E0].T  # noqa: E731
    t = lambda p, q: h[p // 2, q // 2] if p % 2 == q % 2 else 0.0  # noqa: E731
    w = lambda p, q, r, s: eri[p // 2, s // 2, q // 2, r // 2] if p % 2 == s % 2 and q % 2 == r % 2 else 0.0  # noqa: E731
    one, got = np.eye(16), []

    def op(ops, kind, i=-1, j=-1, f=1.0, tr=False):
        if f == 0.0:
            return []
        if (kind, i, j) in ops:
            return [(f, (kind, i, j), tr)]
        return [(f, (kind, j, i), not tr)] if kind in "BQ" and (kind, j, i) in ops else []

    l = lambda *a, **k: op(left_ops, *a, **k)  # noqa: E731
    r = lambda *a, **k: op(right_ops, *a, **k)  # noqa: E731

    def add(x, m, y, both=True):
        if (x is None or x) and (y is None or y) and np.any(m):
            got.append((x, m, y, both))

    add(l("H"), one, None, False)
    add(None, one, r("H"), False)
    A, B = [k[1:] for k in left_ops if k[0] == "A"], [(p, q) for p in X for q in X if l("B", p, q)]
    s = {v: l("S", v) + [e for p in X for e in l("C", p, f=t(p, v))] for v in [*M, *Y]}
    for v in M:
        add(s[v], an(v), None)
        for q in M:
            for z in M:
                if z < v:
                    add([e for p in X for e in l("C", p, f=w(p, q, z, v) - w(p, q, v, z))], cr(q) @ an(z) @ an(v), None)
    for v in Y:
        add(s[v], one, r("C", v, tr=True))
    for p, q in A:
        add(l("A", p, q), one, r("P", p, q))
    for p, q in B:
        if p <= q:
            add(l("B", p, q), one, r("Q", p, q), p < q)
    for p in X:
        add(l("C", p), one, r("U", p))
        for m in M:
            add(l("C", p), cr(m), r("P", p, m))
            add(l("C", p), an(m), r("Q", p, m))
    for m in M:
        for n in M:
            if m < n:
                add([e for p, q in A for e in l("A", p, q, f=w(p, q, m, n) - w(p, q, n, m))], an(m) @ an(n), None)
            if m <= n:
                add([e for p, q in B for e in l("B", p, q, f=w(p, m, n, q) - w(p, m, q, n))], cr(m) @ an(n), None, m < n)
        for v in Y:
            add([e for p, q in A for e in l("A", p, q, f=w(p, q, m, v) - w(p, q, v, m))], an(m), r("C", v, tr=True))
            add([e for p, q in B for e in l("B", p, q, f=w(p, m, v, q) - w(p, m, q, v))], cr(m), r("C", v, tr=True))
            for n in M:
                if m < n:
                    add([e for p in X for e in l("C", p, f=w(p, v, m, n) - w(p, v, n, m))], an(m) @ an(n), r("C", v))
                add([e for p in X for e in l("C", p, f=w(p, m, n, v) - w(p, m, v, n))], cr(m) @ an(n), r("C", v, tr=True))
    for v in Y:
        sv = sum(t(m, v) * cr(m) for m in M) + sum(w(m, n, o, v) * cr(m) @ cr(n) @ an(o) for m in M for n in M for o in M if w(m, n, o, v))
        add(None, sv, r("C", v, tr=True))
    for m in M:
        add(None, cr(m), r("U", m))
        for n in M:
            if m < n:
                add(None, cr(m) @ cr(n), r("P", m, n))
            if m <= n:
                add(None, cr(m) @ an(n), r("Q", m, n), m < n)
    on = sum(t(m, n) * cr(m) @ an(n) for m in M for n in M)
    on = on + 0.5 * sum(w(m, n, o, v) * cr(m) @ cr(n) @ an(o) @ an(v) for m in M for n in M for o in M for v in M if w(m, n, o, v))
    add(None, on, None, False)
    return got


def _summed(terms, dense):
    if terms is None:
        return None
    m = 0.0
    for f, key, tr in terms:
        m = m + f * (dense[key].T if tr else dense[key])
    return m


def _odd(terms):
    return 0 if terms is None else int(terms[0][1][0] in "CSU")


def _apply(case, seed, x):
    """H x in 64 bits: every term as dense matrices over the whole left and right basis."""
    h, eri = _integrals(case["L"], seed)
    site, (left, right) = _blocks(case)
    left.fill(seed + 1), right.fill(seed + 2)
    lay, ld, rd, lp = _layout(case, left, right), left.dense(), right.dense(), left.parity()
    par = torch.tensor(np.diag(_fermions()[1]).copy(), device=DEV)
    psi = torch.zeros(left.start[-1], 16, right.start[-1], dtype=torch.float64, device=DEV)
    y, off = torch.zeros_like(psi), 0
    places = []
    for a, b, c, d in lay:
        n = left.dims[a] * right.dims[d]
        where = (slice(left.start[a], left.start[a + 1]), 4 * b + c, slice(right.start[d], right.start[d + 1]))
        psi[where] = x[off:off + n].view(left.dims[a], right.dims[d])
        places.append((where, off, n))
        off += n
    for lt, m, rt, both in _terms(case["L"], site, h, eri, left.at, right.at):
        po, pr = _odd(lt), _odd(rt)
        pm = (po + pr) % 2
        O, R, S = _summed(lt, ld), _summed(rt, rd), torch.tensor(m, device=DEV)
        if (pm + pr) % 2:
            O = torch.diag(lp) if O is None else O * lp
        if pr:
            S = S * par
        for tr in (False, True) if both else (False,):
            o, s, q = (None if O is None else O.T, S.T, None if R is None else R.T) if tr else (O, S, R)
            to, frm = torch.nonzero(s.abs().sum(1)).view(-1), torch.nonzero(s.abs().sum(0)).view(-1)
            z = psi[:, frm]
            if q is not None:
                z = (z.reshape(-1, z.shape[2]) @ q.T).view(z.shape)
            if o is not None:
                z = (o @ z.reshape(z.shape[0], -1)).view(z.shape)
            y[:, to] += torch.einsum("ij,ajr->air", s[to][:, frm], z)
    out = torch.empty_like(x)
    for where, off, n in places:
        out[off:off + n] = y[where].reshape(-1)
    return out


def _hpsi_work(case):
    """Bytes: every operator block, x and y once. Operations: per term and pair of psi blocks the cheaper
    order of the two products, summed operators counted as one."""
    zero = np.random.RandomState(0)
    L = case["L"]
    h, b = zero.standard_normal((L, L)), zero.standard_normal((2, L, L))
    eri = _Factored(b)
    site, (left, right) = _blocks(case)
    lay, seen, flops = _layout(case, left, right), {}, 0.0
    ma, md = np.array(left.dims), np.array(right.dims)
    src = [[(a, d) for a, b2, c, d in lay if 4 * b2 + c == i] for i in range(16)]
    present = set(lay)
    for lt, m, rt, both in _terms(L, site, h, eri, left.at, right.at):
        dl, dr = (None if t is None else tuple((-1 if t[0][2] else 1) * v for v in _delta(*t[0][1])) for t in (lt, rt))
        key = (dl, dr, (m != 0).tobytes())
        if key not in seen:
            n = 0.0
            for j, i in np.argwhere(m != 0):
                for a, d in src[i]:
                    qa, qd = left.sec[a], right.sec[d]
                    a2 = a if dl is None else left.index.get((qa[0] + dl[0], qa[1] + dl[1]))
                    d2 = d if dr is None else right.index.get((qd[0] + dr[0], qd[1] + dr[1]))
                    if a2 is None or d2 is None or (a2, j // 4, j % 4, d2) not in present:
                        continue
                    if dl is None or dr is None:
                        n += ma[a2] * md[d2] * (0 if dl is None and dr is None else ma[a] if dr is None else md[d])
                    else:
                        n += min(ma[a2] * ma[a] * md[d] + ma[a2] * md[d] * md[d2], ma[a] * md[d] * md[d2] + ma[a2] * ma[a] * md[d2])
            seen[key] = 2.0 * float(n)
        flops += seen[key] * (2 if both else 1)
    n = sum(left.dims[a] * right.dims[d] for a, _, _, d in lay)
    return {"bytes": 8.0 * (left.size + right.size + 2 * n), "flops": flops}


class _Factored:
    """Two-electron integrals kept as factors, read one at a time."""

    def __init__(self, b):
        self.b = b

    def __getitem__(self, i):
        return float(self.b[:, i[0], i[1]] @ self.b[:, i[2], i[3]])


# ------------------------------------------------------------------------------- enlarged blocks
def _enlarged(block):
    """Sectors of block + site, ascending, each with its (block sector, site state) pairs: left blocks
    stand before the site, right blocks after it."""
    got = {}
    order = [(s, a) for s in range(4) for a in range(block.n_sec)] if block.right else [(s, a) for a in range(block.n_sec) for s in range(4)]
    for s, a in order:
        q = (block.sec[a][0] + SITE_QN[s][0], block.sec[a][1] + SITE_QN[s][1])
        got.setdefault(q, []).append((a, s))
    return [(q, got[q], sum(block.dims[a] for a, _ in got[q])) for q in sorted(got)]


def _kept(big, M):
    """How many states each enlarged sector keeps of M in all: more of the larger ones."""
    n = np.array([d for _, _, d in big], dtype=float)
    w = n ** 1.3
    return [int(min(d, round(M * v / w.sum()))) for (_, _, d), v in zip(big, w)]


def _basis(big, kept, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.linalg.qr(torch.randn(d, k, device=DEV, dtype=torch.float64, generator=g))[0] if k else
            torch.zeros(d, 0, device=DEV, dtype=torch.float64) for (_, _, d), k in zip(big, kept)]


def _renorm_plan(case):
    _, (left, _) = _blocks(case, only="H")
    big = _enlarged(left)
    kept, at = _kept(big, case["M"]), {q: i for i, (q, _, _) in enumerate(big)}
    out, inn = [], []
    for k in range(case["ops"]):  # number conserving, one electron more, two more, a spin flip
        d = [(0, 0), (1, 0), (0, 1), (1, 1), (1, -1)][k % 5]
        for i, (q, _, _) in enumerate(big):
            j = at.get((q[0] + d[0], q[1] + d[1]))
            if j is not None:
                out.append(j)
                inn.append(i)
    dims = [d for _, _, d in big]
    off = lambda v: np.concatenate([[0], np.cumsum(v)]).astype(np.int64)  # noqa: E731
    return dict(big=big, dims=dims, kept=kept, out=out, inn=inn, o_off=off([d * k for d, k in zip(dims, kept)]),
                a_off=off([dims[j] * dims[i] for j, i in zip(out, inn)]), r_off=off([kept[j] * kept[i] for j, i in zip(out, inn)]))


def _batch(case):
    r = random.Random(case["n"] * 1000 + case["L0"] * 10 + case["M1"])
    got = []
    for _ in range(case["n"]):
        c = _bond_of(r, case["L0"], case["L1"], case["M0"], case["M1"])
        got.append({**c, "pairs": 0})
    return got


def _grow_in(case, seed):
    site, blocks = _blocks(case)
    block = blocks[case["side"]].fill(seed + 1)
    big = _enlarged(block)
    kept = _kept(big, case["M"])
    return site, block, big, [o.cpu().numpy() for o in _basis(big, kept, seed + 3)]


def _features(n, g):
    f = torch.zeros(n, 16, device=DEV)
    f[:, :4] = torch.asinh(torch.randn(n, 4, device=DEV, generator=g))
    for k in (4, 8):
        f[torch.arange(n, device=DEV), k + torch.randint(0, 4, (n,), device=DEV, generator=g)] = 1.0
    f[:, 12:14] = torch.asinh(torch.rand(n, 2, device=DEV, generator=g))
    f[:, 14:] = torch.rand(n, 2, device=DEV, generator=g) * 0.6
    return f


def _network(seed):
    """Parameters of a network after some training: W1, b1, W2, b2, w3, b3 in the library's order."""
    r = np.random.RandomState(seed % (1 << 31))
    parts = [r.uniform(-1, 1, (16, 256)) * math.sqrt(6 / 16), 0.05 * r.standard_normal(256),
             r.uniform(-1, 1, (256, 256)) * math.sqrt(6 / 256), 0.05 * r.standard_normal(256), 0.02 * r.standard_normal(256),
             0.01 * r.standard_normal(1)]
    return [p.astype(np.float32) for p in parts]


def _pairs(n, g):
    p = torch.randn(n, 3, device=DEV, generator=g)
    p[:, 2] = 1.0
    return p


# ------------------------------------------------------------------------------- prepare and run
def _hop(case, seed, split=False, only=None):
    h, eri = _integrals(case["L"], seed)
    site, (left, right) = _blocks(case, only)
    left.fill(seed + 1), right.fill(seed + 2)
    return dm.Hop(h, eri, left, right, case["na"], case["nb"], site, device=0, want_split=split,
                  share=bool(case.get("pairs") or only))


def _vector(n, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(n, device=DEV, dtype=torch.float64, generator=g)
    return x / x.norm()


def prepare(case, seed):
    kind, seed = case["kind"], 10 * seed
    if kind == "hpsi":
        hop = _hop(case, seed, case["split"])
        x = _vector(hop.n_coeff, seed + 4)
        return dict(kind=kind, hop=hop, x=x, y=torch.empty_like(x), prec=dm.PREC_SPLIT2 if case["split"] else dm.PREC_FP64,
                    graph=case["graph"])
    if kind == "batch":
        hop = dm.Hop.combine([_hop(c, seed + 100 * i, case["split"]) for i, c in enumerate(_batch(case))])
        x = _vector(hop.n_coeff, seed + 4)
        return dict(kind="hpsi", hop=hop, x=x, y=torch.empty_like(x), prec=dm.PREC_SPLIT2 if case["split"] else dm.PREC_FP64,
                    graph=True)
    if kind == "davidson":
        hop = _hop(case, seed)
        return dict(kind=kind, hop=hop, x=_vector(hop.n_coeff, seed + 4), iters=case["iters"])
    if kind == "rdm":
        hop = _hop(case, seed, only="H")
        off = (hop.rdm_right_layout if case["side"] else hop.rdm_left_layout)()[2]
        return dict(kind=kind, hop=hop, x=_vector(hop.n_coeff, seed + 4), side=case["side"],
                    rho=torch.empty(int(off[-1]), device=DEV, dtype=torch.float64))
    if kind == "renorm":
        p, g = _renorm_plan(case), torch.Generator(device=DEV).manual_seed(seed + 1)
        a = torch.randn(int(p["a_off"][-1]), device=DEV, dtype=torch.float64, generator=g)
        o = torch.cat([v.reshape(-1) for v in _basis(p["big"], p["kept"], seed + 3)])
        return dict(kind=kind, plan=p, a=a, o=o, out=torch.empty(int(p["r_off"][-1]), device=DEV, dtype=torch.float64))
    if kind == "grow":
        h, eri = _integrals(case["L"], seed)
        site, block, _, basis = _grow_in(case, seed)
        return dict(kind=kind, args=(h, eri, case["na"], case["nb"], site, block, case["side"]), basis=basis)
    g = torch.Generator(device=DEV).manual_seed(seed + 1)
    net = dm.Mlp(0, seed=1)
    net.set_params(np.concatenate([p.ravel() for p in _network(seed)]))
    s = dict(kind=kind, net=net, feat=_features(case["rows"], g))
    if kind == "mlp_forward":
        return {**s, "out": torch.empty(case["rows"], device=DEV)}
    return {**s, "pairs": _pairs(case["rows"], g), "grad": torch.empty(dm.binding.MLP_PARAMS, device=DEV),
            "loss": torch.empty(1, device=DEV)}


def run(state):
    kind = state["kind"]
    if kind == "hpsi":
        (state["hop"].hpsi_graph if state["graph"] else state["hop"].hpsi)(state["x"], state["y"], state["prec"])
        return state["y"]
    if kind == "davidson":
        psi = state["x"].clone()
        r = state["hop"].davidson(psi, tol=1e-8, max_iter=state["iters"])
        return {"psi": psi, "energy": r["energy"], "resid": r["resid"]}
    if kind == "rdm":
        (state["hop"].rdm_right if state["side"] else state["hop"].rdm_left)(state["x"], state["rho"])
        return state["rho"]
    if kind == "renorm":
        p = state["plan"]
        dm.renormalize_blocks(p["dims"], p["kept"], p["o_off"][:-1], state["o"], p["out"], p["inn"], p["a_off"][:-1], state["a"],
                              p["r_off"][:-1], state["out"])
        return state["out"]
    if kind == "grow":
        grown = dm.block_grow(*state["args"], O=state["basis"])
        data, table = grown.flatten()
        return {"data": data, "dim": grown.dim, "qn": grown.qn, "table": np.array([r for rows in table for r in rows], dtype=np.int64)}
    if kind == "mlp_forward":
        state["net"].forward(state["feat"], state["out"])
        return state["out"]
    state["net"].grad(state["feat"], state["pairs"], state["grad"], state["loss"])
    return {"grad": state["grad"], "loss": state["loss"]}


# ------------------------------------------------------------------------------------- work
def work(case):
    kind = case["kind"]
    if kind == "hpsi":
        return _hpsi_work(case)
    if kind == "batch":
        all_ = [_hpsi_work(c) for c in _batch(case)]
        return {k: sum(w[k] for w in all_) for k in ("bytes", "flops")}
    if kind == "davidson":  # the matvecs, and the basis and its images read for the projections
        one = _hpsi_work(case)
        _, (left, right) = _blocks(case)
        n, m = sum(left.dims[a] * right.dims[d] for a, _, _, d in _layout(case, left, right)), case["iters"]
        return {"bytes": m * one["bytes"] + 8.0 * n * m * (m + 8), "flops": m * one["flops"] + 8.0 * n * m * m}
    if kind == "rdm":
        _, (left, right) = _blocks(case, only="H")
        lay = _layout(case, left, right)
        me, n, groups, flops = (left, right)[case["side"]], 0, {}, 0.0
        for a, b, c, d in lay:  # row groups (sector of the enlarged block) by the columns that they share
            (sec, st), other = ((a, b), (c, d)) if case["side"] == 0 else ((d, c), (b, a))
            cols = right.dims[d] if case["side"] == 0 else left.dims[a]
            q = (me.sec[sec][0] + SITE_QN[st][0], me.sec[sec][1] + SITE_QN[st][1])
            groups.setdefault((q, other), []).append((me.dims[sec], cols))
            n += left.dims[a] * right.dims[d]
        for g in groups.values():  # rho is symmetric: half of the products
            flops += float(sum(r for r, _ in g) ** 2 * g[0][1])
        return {"bytes": 8.0 * (n + sum(dim * dim for _, _, dim in _enlarged(me))), "flops": flops}
    if kind == "renorm":
        p = _renorm_plan(case)
        dims, k = p["dims"], p["kept"]
        flops = sum(2.0 * min(dims[j] * dims[i] * k[i] + dims[j] * k[j] * k[i], dims[j] * dims[i] * k[j] + dims[i] * k[j] * k[i])
                    for j, i in zip(p["out"], p["inn"]))
        return {"bytes": 8.0 * float(p["a_off"][-1] + p["r_off"][-1] + p["o_off"][-1]), "flops": flops}
    if kind == "grow":
        block = _blocks(case)[1][case["side"]]
        big = _enlarged(block)
        kept = dict(zip([q for q, _, _ in big], _kept(big, case["M"])))
        grown = flops = 0.0
        for o in block.ops:  # O_out^T Z O_in for the identity on the site: every old operator goes on
            d = _delta(o.kind, o.i0, o.i1)
            for so, si, _ in o.rows:
                for s in SITE_QN:
                    ko, ki = (kept[(block.sec[v][0] + s[0], block.sec[v][1] + s[1])] for v in (so, si))
                    flops += 2.0 * (block.dims[so] * block.dims[si] * ki + block.dims[so] * ko * ki)
            grown += sum(kept[q] * kept.get((q[0] + d[0], q[1] + d[1]), 0) for q in kept)
        return {"bytes": 8.0 * (block.size + grown), "flops": flops}
    n = float(case["rows"])
    one = 2.0 * n * (16 * 256 + 256 * 256 + 256)
    if kind == "mlp_forward":
        return {"bytes": 4 * n * 17 + 2.0 * 70000, "flops": one}
    return {"bytes": 4 * n * 19 + 8.0 * 70000, "flops": 3 * one}


# ------------------------------------------------------------------------------------- exact
def exact(case, seed):
    kind, seed = case["kind"], 10 * seed
    if kind == "hpsi":
        if case["pairs"] or case["M"] * case["M"] * case["L"] ** 2 > 7e8:
            return None  # too large to do densely
        return _apply(case, seed, _vector(_count(case), seed + 4))
    if kind == "batch":
        parts = _batch(case)
        x, got, at = _vector(sum(_count(c) for c in parts), seed + 4), [], 0
        for i, c in enumerate(parts):
            n = _count(c)
            got.append(_apply(c, seed + 100 * i, x[at:at + n].contiguous()))
            at += n
        return torch.cat(got)
    if kind == "davidson":
        return None  # sixteen steps of an unconverged solve: no value but the method's own
    if kind == "rdm":
        _, blocks = _blocks(case, only="H")
        me, lay = blocks[case["side"]], _layout(case, *blocks)
        x, at, parts = _vector(_count(case), seed + 4), 0, {}
        for a, b, c, d in lay:
            n = blocks[0].dims[a] * blocks[1].dims[d]
            m = x[at:at + n].view(blocks[0].dims[a], blocks[1].dims[d])
            parts.setdefault((c, d) if case["side"] == 0 else (a, b), {})[(a, b) if case["side"] == 0 else (d, c)] = m if case["side"] == 0 else m.T
            at += n
        got = []
        for q, pairs, dim in _enlarged(me):
            rho, place, pos = torch.zeros(dim, dim, dtype=torch.float64, device=DEV), {}, 0
            for p in pairs:
                place[p] = slice(pos, pos + me.dims[p[0]])
                pos += me.dims[p[0]]
            for group in parts.values():
                if next(iter(group)) in place:
                    for p, u in group.items():
                        for s, v in group.items():
                            rho[place[p], place[s]] += u @ v.T
            got.append(rho.reshape(-1))
        return torch.cat(got)
    if kind == "renorm":
        p, g = _renorm_plan(case), torch.Generator(device=DEV).manual_seed(seed + 1)
        a = torch.randn(int(p["a_off"][-1]), device=DEV, dtype=torch.float64, generator=g)
        o = _basis(p["big"], p["kept"], seed + 3)
        return torch.cat([(o[j].T @ a[p["a_off"][n]:p["a_off"][n + 1]].view(p["dims"][j], p["dims"][i]) @ o[i]).reshape(-1)
                          for n, (j, i) in enumerate(zip(p["out"], p["inn"]))])
    if kind == "grow":
        return {"data": _grown_left(case, seed) if case["side"] == 0 else None, "dim": None, "qn": None, "table": None}
    g = torch.Generator(device=DEV).manual_seed(seed + 1)
    f = _features(case["rows"], g).double()
    w1, b1, w2, b2, w3, b3 = [torch.tensor(p, device=DEV, dtype=torch.float64) for p in _network(seed)]
    h1 = torch.relu(f @ w1 + b1)
    h2 = torch.relu(h1 @ w2 + b2)
    m = h2 @ w3 + b3
    if kind == "mlp_forward":
        return m
    a, b, wt = _pairs(case["rows"], g).double().unbind(1)
    e = a * (1 + m) - b
    dm_ = 2 * wt * a * e / case["rows"]
    d2 = dm_[:, None] * w3 * (h2 > 0)
    d1 = (d2 @ w2.T) * (h1 > 0)
    grad = [f.T @ d1, d1.sum(0), h1.T @ d2, d2.sum(0), h2.T @ dm_, dm_.sum()[None]]
    return {"grad": torch.cat([v.reshape(-1) for v in grad]), "loss": (wt * e * e).mean()[None]}


def _count(case):
    _, (left, right) = _blocks(case, only="H")
    return sum(left.dims[a] * right.dims[d] for a, _, _, d in _layout(case, left, right))


def _grown_left(case, seed):
    """The normal operators of a left block grown by its site, from their definitions, in the basis O."""
    h, eri = _integrals(case["L"], seed)
    site, block, big, basis = _grow_in(case, seed)
    old, par, n = block.dense(), torch.diag(block.parity()), int(block.start[-1])
    X, s, W = range(2 * site), (2 * site, 2 * site + 1), range(2 * site + 2, 2 * case["L"])
    up, down, one = torch.zeros(4, 4), torch.zeros(4, 4), torch.eye(4, dtype=torch.float64, device=DEV)
    up[1, 0] = up[3, 2] = down[2, 0] = 1.0
    down[3, 1] = -1.0
    cr = dict(zip(s, (up.double().to(DEV), down.double().to(DEV))))
    t = lambda p, q: h[p // 2, q // 2] if p % 2 == q % 2 else 0.0  # noqa: E731
    w = lambda p, q, r, v: eri[p // 2, v // 2, q // 2, r // 2] if p % 2 == v % 2 and q % 2 == r % 2 else 0.0  # noqa: E731
    B = lambda p, q: old[("B", p, q)] if p <= q else old[("B", q, p)].T  # noqa: E731
    none = torch.zeros(n, n, dtype=torch.float64, device=DEV)
    lift = lambda m, x, odd: torch.kron((m @ par if odd else m).contiguous(), x.contiguous())  # noqa: E731
    zero, eye = torch.zeros(4, 4, dtype=torch.float64, device=DEV), torch.eye(n, dtype=torch.float64, device=DEV)
    H = lift(old[("H", -1, -1)], one, 0)
    hs = sum((t(p, q) * cr[p] @ cr[q].T for p in s for q in s), zero)
    hs = hs + 0.5 * sum((w(p, q, r, v) * cr[p] @ cr[q] @ cr[r].T @ cr[v].T for p in s for q in s for r in s for v in s), zero)
    H = H + lift(eye, hs, 0)
    cross = torch.zeros_like(H)
    for v in s:
        cross += lift(old[("S", v, -1)] + sum((t(p, v) * old[("C", p, -1)] for p in X), none), cr[v].T, 1)
    for p in X:
        cross += lift(old[("C", p, -1)], sum((w(p, q, z, v) * cr[q] @ cr[z].T @ cr[v].T for q in s for z in s for v in s), zero), 1)
        for q in X:
            if p < q:
                cross += lift(old[("A", p, q)], sum((w(p, q, z, v) * cr[z].T @ cr[v].T for z in s for v in s), zero), 0)
            H = H + lift(B(p, q), sum(((w(p, z, v, q) - w(p, z, q, v)) * cr[z] @ cr[v].T for z in s for v in s), zero), 0)
    new = {("H", -1, -1): H + cross + cross.T}
    c = {p: lift(old[("C", p, -1)], one, 0) for p in X}
    c.update({y: lift(eye, cr[y], 1) for y in s})
    every = [*X, *s]
    new.update({("C", p, -1): c[p] for p in every})
    for kind in "AB":
        for p in every:
            for q in every:
                if p < q or (p == q and kind == "B"):
                    new[(kind, p, q)] = lift(old[(kind, p, q)], one, 0) if q in X else c[p] @ (c[q] if kind == "A" else c[q].T)
    for v in W:
        S = lift(old[("S", v, -1)], one, 0)
        for y in s:
            S = S + lift(sum(((w(p, q, y, v) - w(q, p, y, v)) * old[("A", p, q)] for p in X for q in X if p < q), none), cr[y].T, 1)
            S = S + lift(sum(((w(y, p, q, v) - w(p, y, q, v)) * B(p, q) for p in X for q in X), none), cr[y], 1)
            for z in s:
                S = S + lift(sum(((w(p, y, z, v) - w(y, p, z, v)) * old[("C", p, -1)] for p in X), none), cr[y] @ cr[z].T, 0)
                S = S + lift(sum((w(y, z, q, v) * old[("C", q, -1)].T for q in X), none), cr[y] @ cr[z], 0)
                for r in s:
                    S = S + lift(eye, w(y, z, r, v) * cr[y] @ cr[z] @ cr[r].T, 1)
        new[("S", v, -1)] = S
    rows = [torch.tensor([(block.start[a] + i) * 4 + st for a, st in pairs for i in range(block.dims[a])], device=DEV) for _, pairs, _ in big]
    basis = [torch.from_numpy(o).to(DEV) for o in basis]
    live = [i for i, o in enumerate(basis) if o.shape[1]]
    at, got = {big[i][0]: i for i in live}, []
    for (kind, p, q), m in new.items():
        d, found = _delta(kind, p, q), []
        for i in live:
            j = at.get((big[i][0][0] + d[0], big[i][0][1] + d[1]))
            if j is not None:
                found.append((j, i))
        got += [(basis[j].T @ m[rows[j]][:, rows[i]] @ basis[i]).reshape(-1) for j, i in sorted(found)]
    return torch.cat(got)
