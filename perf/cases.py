"""Work that users of the library have it do, as cases that can be timed and compared.

Every case goes through the public binding (`paper_2609_09990_amd`) with seeded synthetic
inputs: random active-space integrals (a ramp of orbital energies, normal couplings, symmetric
Cholesky vectors), block-sparse random MPS and two-site vectors in the documented slab layout,
random CI vectors and network inputs.  A case is a dict of plain values whose "op" says which
call it stands for:

  sigma     H_eff psi of one two-site step (the inner product of every Davidson iteration), in
            fp64 ("prec" 0) or in the low-precision forms fp32 (1) and bf16 (2)
  truncate  decimation of a two-site state: density matrices, eigensolve, new site tensors and
            environment update, once moving right and once moving left
  sweep     a whole small DMRG run: new solver, sweeps from its seeded start, MPS energy
  grad      energy of a given MPS and its gradient with respect to the integrals (the backward
            of the energy node): every environment of the chain, then the contractions
  rdm12     one- and two-body densities of a CI vector
  rdm3      transition three-body densities of two CI vectors
  apply_v   the two-electron operator on a CI vector
  train     loss and parameter gradient of the preconditioner network on a batch of triples

`exact` computes the same numbers in float64 from the definitions (Fock space with Jordan-Wigner
signs, string tables, plain linear algebra), for the sizes where that is quick.
"""
import math

import numpy as np
import torch

import paper_2609_09990_amd as pk

SITE_QN = ((0, 0), (1, 1), (1, -1), (2, 0))


# ---------------------------------------------------------------- cases --

def listed():
    return [
        # a product in a small active space, where launches and latency count: CAS(8,8), ragged bond
        {"name": "sigma cas8 m60 fp64", "op": "sigma", "n": 8, "na": 4, "nb": 4, "nq": 16, "M": 60, "k": 3, "prec": 0},
        # an ordinary production size: CAS(12,12) at M = 512, middle bond
        {"name": "sigma cas12 m512 fp64", "op": "sigma", "n": 12, "na": 6, "nb": 6, "nq": 64, "M": 512, "k": 5,
         "prec": 0},
        # the benchmark's active space and bond dimension, middle bond: the largest product
        {"name": "sigma cas20 m1024 fp64", "op": "sigma", "n": 20, "na": 10, "nb": 10, "nq": 120, "M": 1024, "k": 9,
         "prec": 0},
        # the precision form's products: fp32 and bf16 on CAS(16,16) at M = 512
        {"name": "sigma cas16 m512 fp32", "op": "sigma", "n": 16, "na": 8, "nb": 8, "nq": 96, "M": 512, "k": 7,
         "prec": 1},
        {"name": "sigma cas16 m512 bf16", "op": "sigma", "n": 16, "na": 8, "nb": 8, "nq": 96, "M": 512, "k": 7,
         "prec": 2},
        # decimation of an ordinary step, both directions: CAS(16,16) at M = 512
        {"name": "truncate cas16 m512", "op": "truncate", "n": 16, "na": 8, "nb": 8, "nq": 96, "M": 512, "k": 7},
        # a whole small run: CAS(8,8), truncated bond, two sweeps
        {"name": "sweep cas8 m64", "op": "sweep", "n": 8, "na": 4, "nb": 4, "nq": 32, "M": 64, "sweeps": 2},
        # the adjoint of an energy: CAS(12,12) at M = 256
        {"name": "grad cas12 m256", "op": "grad", "n": 12, "na": 6, "nb": 6, "nq": 64, "M": 256},
        # densities of a CAS(12,12) CI vector (orbital optimisation, properties)
        {"name": "rdm12 cas12", "op": "rdm12", "n": 12, "na": 6, "nb": 6},
        # three-body densities for the perturbative correction: CAS(10,10)
        {"name": "rdm3 cas10", "op": "rdm3", "n": 10, "na": 5, "nb": 5},
        # the two-electron operator on a CI vector with an odd electron count: CAS(11,12)
        {"name": "apply_v cas12", "op": "apply_v", "n": 12, "na": 6, "nb": 5, "nq": 64},
        # one training step's loss and gradient: 64 triples of 1024 amplitudes
        {"name": "train 64x1024", "op": "train", "segs": 64, "len": 1024, "width": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; sizes are drawn over the whole range, odd ones among them."""
    op = rng.choice(["sigma", "sigma", "sigma", "sigma", "truncate", "sweep", "grad", "rdm12", "rdm3", "apply_v",
                     "train"])
    if op == "sigma":
        n = rng.randint(6, 18)
        na = n // 2
        nb = na - rng.choice([0, 0, 1])
        return {"op": op, "n": n, "na": na, "nb": nb, "nq": rng.randint(2 * n, 6 * n), "M": _log(rng, 16, 800),
                "k": rng.randint(max(0, n // 2 - 3), min(n - 2, n // 2 + 1)), "prec": rng.choice([0, 0, 1, 2])}
    if op == "truncate":
        n = rng.randint(8, 16)
        return {"op": op, "n": n, "na": n // 2, "nb": n // 2 - rng.choice([0, 1]), "nq": rng.randint(2 * n, 6 * n),
                "M": _log(rng, 24, min(512, 4 ** (n // 2) // 3)), "k": n // 2 - rng.choice([1, 2])}
    if op == "sweep":
        n = rng.randint(5, 8)
        return {"op": op, "n": n, "na": (n + 1) // 2, "nb": n // 2, "nq": rng.randint(8, 4 * n),
                "M": rng.randint(16, 64), "sweeps": rng.choice([1, 2])}
    if op == "grad":
        n = rng.randint(6, 12)
        return {"op": op, "n": n, "na": n // 2, "nb": n // 2 - rng.choice([0, 1]), "nq": rng.randint(n, 5 * n),
                "M": _log(rng, 16, 256)}
    if op == "rdm12":
        n = rng.randint(6, 12)
        return {"op": op, "n": n, "na": n // 2, "nb": rng.choice([n // 2, n // 2 - 1])}
    if op == "rdm3":
        n = rng.randint(4, 9)
        return {"op": op, "n": n, "na": (n + 1) // 2, "nb": n // 2}
    if op == "apply_v":
        n = rng.randint(6, 12)
        return {"op": op, "n": n, "na": n // 2, "nb": max(1, n // 2 - rng.choice([1, 2])), "nq": rng.randint(n, 60)}
    return {"op": op, "segs": rng.randint(8, 64), "len": _log(rng, 100, 1024), "width": rng.choice([64, 128, 256, 256])}


# --------------------------------------------------------------- inputs --

def _integrals(n, nq, rng):
    h = np.diag(np.linspace(-2.0, 1.0, n))
    g = np.triu(rng.normal(0.0, 0.05, (n, n)), 1)
    c = np.triu(rng.normal(0.0, 0.1, (nq, n, n)))
    return h + g + g.T, c + np.transpose(np.triu(c, 1), (0, 2, 1))


def _bonds(n, na, nb, M):
    """Sector tables (N, 2S_z, dim) of every cut, full dimensions scaled down to about M states."""
    out = []
    for c in range(n + 1):
        full = []
        for a in range(min(c, na) + 1):
            for b in range(min(c, nb) + 1):
                if na - a <= n - c and nb - b <= n - c:
                    d = min(math.comb(c, a) * math.comb(c, b),
                            math.comb(n - c, na - a) * math.comb(n - c, nb - b))
                    full.append((a + b, a - b, d))
        full.sort()
        tot = sum(d for _, _, d in full)
        out.append(full if tot <= M else [(N, s, max(1, d * M // tot)) for N, s, d in full])
    return out


def _phys(sites):
    if sites == 1:
        return SITE_QN
    return tuple((a[0] + b[0], a[1] + b[1]) for a in SITE_QN for b in SITE_QN)


def _slabs(left, right, sites):
    """Per left sector: rows, [(physical index, right sector index, columns)]."""
    at = {(N, s): j for j, (N, s, _) in enumerate(right)}
    out = []
    for N, s, ml in left:
        cols = [(p, at[(N + dn, s + ds)]) for p, (dn, ds) in enumerate(_phys(sites)) if (N + dn, s + ds) in at]
        out.append((ml, [(p, j, right[j][2]) for p, j in cols]))
    return out


def _mps(case, rng):
    bonds = _bonds(case["n"], case["na"], case["nb"], case["M"])
    sites = []
    for k in range(case["n"]):
        parts = [rng.normal(0.0, 1.0 / math.sqrt(max(1, sum(c[2] for c in cols))), ml * sum(c[2] for c in cols))
                 for ml, cols in _slabs(bonds[k], bonds[k + 1], 1)]
        sites.append(np.concatenate(parts))
    return bonds, sites


def _two_site(bonds, k, rng, decay=None):
    """Normalised two-site vector; with `decay`, rows and columns of every block fall off, as the
    Schmidt weights of a DMRG state do."""
    parts = []
    for ml, cols in _slabs(bonds[k], bonds[k + 2], 2):
        row = [rng.normal(0.0, 1.0, (ml, w)) for _, _, w in cols]
        if decay:
            row = [x * np.exp(-decay * np.arange(ml) / ml)[:, None] * np.exp(-decay * np.arange(x.shape[1]) / x.shape[1])
                   for x in row]
        parts.append(np.concatenate(row, axis=1).ravel() if row else np.zeros(0))
    v = np.concatenate(parts)
    return v / np.linalg.norm(v)


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    op, x = case["op"], {}
    if op == "train":
        n = case["segs"] * case["len"]
        x["X"] = rng.normal(0.0, 1.0, (n, 8)).astype(np.float32)
        x["T"] = (0.5 * x["X"][:, 3] + rng.normal(0.0, 0.5, n)).astype(np.float32)
        w = case["width"]
        x["P"] = {"W1": rng.normal(0, 0.5, (w, 8)), "b1": rng.normal(0, 0.1, w),
                  "W2": rng.normal(0, math.sqrt(2.0 / w), (w, w)), "b2": rng.normal(0, 0.1, w),
                  "W3": rng.normal(0, 1 / math.sqrt(w), (1, w)), "b3": rng.normal(0, 0.1, 1)}
        x["P"] = {k: v.astype(np.float32) for k, v in x["P"].items()}
        return x
    x["h"], x["B"] = _integrals(case["n"], case.get("nq", 4), rng)
    if op in ("rdm12", "rdm3", "apply_v"):
        dims = (math.comb(case["n"], case["na"]), math.comb(case["n"], case["nb"]))
        for name in ("c", "d") if op == "rdm3" else ("c",):
            v = rng.normal(0.0, 1.0, dims)
            x[name] = v / np.linalg.norm(v)
    elif op != "sweep":
        x["bonds"], x["sites"] = _mps(case, rng)
        if op != "grad":
            x["psi"] = _two_site(x["bonds"], case["k"], rng, 10.0 if op == "truncate" else None)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    op = case["op"]
    s = {"case": case, "op": op}
    if op == "train":
        s["X"], s["T"] = torch.from_numpy(x["X"]).cuda(), torch.from_numpy(x["T"]).cuda()
        s["net"] = pk.MLP(8, case["width"])
        s["net"].set_params(pk.MLP.pack(x["P"]))
        return s
    s["prob"] = pk.Problem(x["h"], x["B"], case["na"], case["nb"])
    if op in ("rdm12", "rdm3", "apply_v"):
        for name in ("c", "d"):
            if name in x:
                s[name] = torch.from_numpy(x[name]).cuda()
    elif op == "sweep":
        s["seed"] = 1 + seed % 1000003
    else:
        s["sol"] = pk.Solver(s["prob"], M=case["M"])
        s["sol"].set_mps(x["bonds"], x["sites"])
        if op == "grad":
            s["bonds"], s["sites"] = x["bonds"], x["sites"]
        else:
            s["psi"] = torch.from_numpy(x["psi"]).cuda()
            s["sol"].prepare(case["k"])
        if op == "sigma":
            s["out"] = torch.zeros_like(s["psi"])
    return s


def run(s):
    case, op = s["case"], s["op"]
    if op == "sigma":
        s["sol"].sigma(case["k"], s["psi"], s["out"], case["prec"])
        return {"sigma": s["out"]}
    if op == "truncate":
        out = {}
        for d, name in ((0, "right"), (1, "left")):
            tau, sv = s["sol"].truncate(case["k"], s["psi"], d)
            out[name] = {"tau": tau, "sv": sv}
        return out
    if op == "sweep":
        sol = pk.Solver(s["prob"], M=case["M"], tol=1e-9, seed=s["seed"])
        e, _, _ = sol.sweep(case["sweeps"])
        return {"ritz": e, "mps": sol.energy()}
    if op == "grad":
        s["sol"].set_mps(s["bonds"], s["sites"])
        e = s["sol"].energy()
        dh, dB, _ = s["sol"].grad()
        return {"energy": e, "dh": dh, "dB": dB}
    if op == "rdm12":
        g, G, _ = s["prob"].ci_rdm12(s["c"])
        return {"gamma": g, "Gamma": G}
    if op == "rdm3":
        return {"rdm3": s["prob"].ci_rdm3(s["c"], s["d"])}
    if op == "apply_v":
        return {"Vc": s["prob"].ci_apply_v(s["c"])}
    loss, grad = s["net"].loss_grad(s["X"], s["T"], case["segs"], case["len"], want_grad=True)
    return {"loss": loss, "grad": grad}


# ----------------------------------------------------------------- work --

def work(case):
    """Bytes and operations of one pass by its definition: inputs read and outputs written once; for
    the products of the chain, one product with every operator channel on either side of a bond (an
    estimate from the sector tables: a density channel per Cholesky vector, two one-fermion channels
    per orbital and spin, and the pair channels of the smaller side)."""
    op = case["op"]
    if op == "train":
        rows, w = case["segs"] * case["len"], case["width"]
        return {"bytes": 4.0 * (rows * 9 + 2 * (w * w + 11 * w)), "flops": 6.0 * rows * w * (w + 8 + 1)}
    n = case["n"]
    if op in ("rdm12", "rdm3", "apply_v"):
        det = math.comb(n, case["na"]) * math.comb(n, case["nb"])
        n2 = n * n
        if op == "rdm12":
            return {"bytes": 8.0 * (det + n2 * n2 + n2), "flops": 1.0 * n2 * (n2 + 1) * det}
        if op == "rdm3":
            return {"bytes": 8.0 * (2 * det + n2 ** 3), "flops": 2.0 * n2 * n2 * n2 * det}
        return {"bytes": 16.0 * det, "flops": 4.0 * case["nq"] * n2 * det}
    bonds = _bonds(n, case["na"], case["nb"], case["M"])

    def step(k):
        """Environment elements and product flops of one H_eff product at sites (k, k + 1)."""
        half = min(k + 1, n - k - 1)
        shifts = [((0, 0), 2 + case["nq"])] + [(q, n) for q in ((1, 1), (1, -1), (-1, 1), (-1, -1))]
        shifts += [(q, half * half // 2) for q in ((0, 2), (0, -2), (2, 0), (-2, 0))]
        dl, dr = ({(N, q): d for N, q, d in bonds[c]} for c in (k, k + 2))
        wl, wr = {}, {}  # two-site columns of every left sector, rows of every right sector
        for (N, q, ml), (_, cols) in zip(bonds[k], _slabs(bonds[k], bonds[k + 2], 2)):
            wl[N, q] = sum(c[2] for c in cols)
            for _, j, _ in cols:
                wr[bonds[k + 2][j][:2]] = wr.get(bonds[k + 2][j][:2], 0) + ml
        size = sum(dl[q] * w for q, w in wl.items())
        env, fl = 0, 0.0
        for (dn, ds), count in shifts:
            for d, w in ((dl, wl), (dr, wr)):
                for (N, q), m in d.items():
                    out = d.get((N + dn, q + ds), 0)
                    env += count * m * out
                    fl += 2.0 * count * m * out * w.get((N, q), 0)
        return size, env, fl

    if op == "sigma":
        size, env, fl = step(case["k"])
        return {"bytes": 16.0 * size + (8, 4, 2)[case["prec"]] * env, "flops": fl}
    if op == "truncate":
        size, env, fl = step(case["k"])
        return {"bytes": 2 * 8.0 * (2 * size + env), "flops": 0.5 * fl + 40.0 * case["M"] * size}
    all_steps = [step(k) for k in range(n - 1)]
    env, fl = sum(x[1] for x in all_steps), sum(x[2] for x in all_steps)
    if op == "sweep":
        return {"bytes": 2.0 * case["sweeps"] * 8 * env, "flops": 2.0 * case["sweeps"] * 10 * fl}
    return {"bytes": 8.0 * 2 * env, "flops": 2.0 * fl}


# ---------------------------------------------------------------- exact --

def _dense(left, right, sites, flat):
    """Dense [D_left, 4^sites, D_right] tensor of a slab-layout tensor."""
    lo = np.concatenate([[0], np.cumsum([d for _, _, d in left])])
    ro = np.concatenate([[0], np.cumsum([d for _, _, d in right])])
    t, at = np.zeros((lo[-1], 4 ** sites, ro[-1])), 0
    where = np.zeros(len(flat), dtype=np.int64)
    for i, (ml, cols) in enumerate(_slabs(left, right, sites)):
        w = sum(c[2] for c in cols)
        block, col = where[at:at + ml * w].reshape(ml, w), 0
        for p, j, m in cols:
            r = np.arange(lo[i], lo[i] + ml)[:, None]
            c = np.arange(ro[j], ro[j] + m)[None, :]
            block[:, col:col + m] = (r * t.shape[1] + p) * t.shape[2] + c
            col += m
        at += ml * w
    t.reshape(-1)[where] = flat
    return t, where


def _products(bonds, sites, k0, k1):
    """[D_{k0}, 4^(k1 - k0), D_{k1}] product of the site tensors k0 .. k1 - 1 (first site slowest)."""
    out = torch.eye(sum(d for _, _, d in bonds[k0]), dtype=torch.float64).cuda()[:, None, :]
    for k in range(k0, k1):
        a = torch.from_numpy(_dense(bonds[k], bonds[k + 1], 1, sites[k])[0]).cuda()
        out = torch.matmul(out.reshape(-1, a.shape[0]), a.reshape(a.shape[0], -1))
        out = out.reshape(sum(d for _, _, d in bonds[k0]), -1, a.shape[2])
    return out


class _Fock:
    """Excitations E_pq on the determinants of one (n_alpha, n_beta) sector, Jordan-Wigner order
    0a, 0b, 1a, 1b, ...; flat index of a state: site 0 slowest, s = n_alpha + 2 n_beta per site."""

    def __init__(self, n, na, nb):
        idx = torch.arange(4 ** n, device="cuda")
        occ = torch.zeros_like(idx)
        for k in range(n):
            occ |= ((idx >> (2 * (n - 1 - k))) & 3) << (2 * k)
        alpha = sum((occ >> (2 * k)) & 1 for k in range(n))
        beta = sum((occ >> (2 * k + 1)) & 1 for k in range(n))
        self.index = torch.nonzero((alpha == na) & (beta == nb)).reshape(-1)  # flat index of each determinant
        self.occ, self.n = occ[self.index], n
        self.row = torch.full((4 ** n,), -1, dtype=torch.int64, device="cuda")
        self.row[self.occ] = torch.arange(len(self.occ), device="cuda")
        self.table = {}
        for p in range(n):
            for q in range(n):
                self.table[p, q] = [self._hop(2 * p + s, 2 * q + s) for s in (0, 1)]

    def _parity(self, x):
        for sh in (16, 8, 4, 2, 1):
            x = x ^ (x >> sh)
        return (x & 1).double()

    def _hop(self, i, j):
        """Rows from, rows to and signs of a+_i a_j."""
        o = self.occ
        ok = ((o >> j) & 1) == 1
        if i != j:
            ok &= ((o >> i) & 1) == 0
        src = torch.nonzero(ok).reshape(-1)
        o = o[src]
        mid = o & ~(1 << j)
        sign = 1 - 2 * ((self._parity(o & ((1 << j) - 1)) + self._parity(mid & ((1 << i) - 1))) % 2)
        return src, self.row[mid | (1 << i)], sign

    def excite(self, p, q, c):
        out = torch.zeros_like(c)
        for src, dst, sign in self.table[p, q]:
            out.index_add_(0, dst, sign * c[src])
        return out

    def all(self, c):
        return torch.stack([self.excite(p, q, c) for p in range(self.n) for q in range(self.n)])

    def apply_h(self, h, B, c):
        h, B = torch.from_numpy(h).cuda(), torch.from_numpy(B).cuda()
        n = self.n
        T = self.all(c)
        # 1/2 sum (pq|rs)(E_pq E_rs - d_qr E_ps)
        one = h - 0.5 * torch.matmul(B.permute(1, 0, 2).reshape(n, -1), B.permute(0, 1, 2).reshape(-1, n))
        out = torch.matmul(one.reshape(-1), T)
        F = B.reshape(B.shape[0], -1)
        U = torch.matmul(F.t().contiguous(), torch.matmul(F, T))
        for p in range(n):
            for q in range(n):
                out += 0.5 * self.excite(p, q, U[p * n + q])
        return out


def _strings(n, k):
    m = np.arange(1 << n)
    pop = np.array([bin(x).count("1") for x in m])
    return m[pop == k]


def _string_hop(n, strs, r, s):
    """E_rs on one spin's strings: rows from, rows to, signs."""
    row = np.full(1 << n, -1)
    row[strs] = np.arange(len(strs))
    ok = (strs >> s & 1) == 1
    if r != s:
        ok &= (strs >> r & 1) == 0
    src = np.nonzero(ok)[0]
    o = strs[src]
    mid = o & ~(1 << s)
    pop = np.array([bin(x).count("1") for x in range(1 << n)])
    sign = 1.0 - 2.0 * ((pop[o & ((1 << s) - 1)] + pop[mid & ((1 << r) - 1)]) % 2)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    return to(src), to(row[mid | (1 << r)]), to(sign)


class _CI:
    """E_rs on CI matrices c[alpha string][beta string] (strings ascending, alpha operators first)."""

    def __init__(self, n, na, nb):
        a, b = _strings(n, na), _strings(n, nb)
        self.n = n
        self.hops = [(_string_hop(n, a, r, s), _string_hop(n, b, r, s)) for r in range(n) for s in range(n)]

    def excite(self, x, c):
        (si, di, gi), (sj, dj, gj) = self.hops[x]
        out = torch.zeros_like(c)
        out[di] += gi[:, None] * c[si]
        out[:, dj] += gj[None, :] * c[:, sj]
        return out

    def all(self, c):
        return torch.stack([self.excite(x, c).reshape(-1) for x in range(self.n * self.n)])


def _network(P, X, T, segs, length):
    P = {k: torch.from_numpy(v).double().cuda().requires_grad_() for k, v in P.items()}
    x, t = torch.from_numpy(X).double().cuda(), torch.from_numpy(T).double().cuda().reshape(segs, length)
    a = torch.relu(torch.matmul(x, P["W1"].t()) + P["b1"])
    a = torch.relu(torch.matmul(a, P["W2"].t()) + P["b2"])
    y = (torch.matmul(a, P["W3"].t()) + P["b3"]).reshape(segs, length)
    loss = (1.0 - (y * t).sum(1) / (y.norm(dim=1) * t.norm(dim=1))).mean()
    loss.backward()
    grad = torch.cat([P[k].grad.reshape(-1) for k in ("W1", "b1", "W2", "b2", "W3", "b3")])
    return {"loss": float(loss), "grad": grad}


def _schmidt(case, x):
    """Singular values of the two-site state across its middle bond, descending."""
    bl, br = x["bonds"][case["k"]], x["bonds"][case["k"] + 2]
    t, _ = _dense(bl, br, 2, x["psi"])
    t = torch.from_numpy(t).cuda().reshape(t.shape[0], 4, 4, t.shape[2])
    values = []
    qn_l = torch.tensor([[N, q] for N, q, d in bl for _ in range(d)]).cuda()
    qn_r = torch.tensor([[N, q] for N, q, d in br for _ in range(d)]).cuda()
    phys = torch.tensor(SITE_QN).cuda()
    rows = (qn_l[:, None, :] + phys[None, :, :]).reshape(-1, 2)
    cols = (qn_r[None, :, :] - phys[:, None, :]).reshape(-1, 2)
    full = t.reshape(rows.shape[0], cols.shape[0])
    for q in torch.unique(rows, dim=0):
        block = full[(rows == q).all(1)][:, (cols == q).all(1)]
        if block.numel():
            values.append(torch.linalg.svdvals(block))
    return torch.sort(torch.cat(values), descending=True).values


def exact(case, seed):
    op = case["op"]
    if op == "sweep" or (op in ("sigma", "grad") and case["n"] > 10):
        return None
    x = _inputs(case, seed)
    if op == "train":
        return _network(x["P"], x["X"], x["T"], case["segs"], case["len"])
    n = case["n"]
    if op == "truncate":
        s = _schmidt(case, x)
        keep = min(case["M"], len(s))
        one = {"tau": float((s[keep:] ** 2).sum()), "sv": s[:keep]}
        return {"right": one, "left": one}
    if op in ("rdm12", "rdm3", "apply_v"):
        ci = _CI(n, case["na"], case["nb"])
        c = torch.from_numpy(x["c"]).cuda()
        T = ci.all(c)
        flip = torch.arange(n * n).reshape(n, n).t().reshape(-1).cuda()  # row pq of E_qp
        if op == "apply_v":
            F = torch.from_numpy(x["B"]).cuda().reshape(-1, n * n)
            U = torch.matmul(F.t().contiguous(), torch.matmul(F, T))
            return {"Vc": sum(0.5 * ci.excite(y, U[y].reshape(c.shape)) for y in range(n * n))}
        if op == "rdm12":
            gamma = torch.matmul(T, c.reshape(-1)).reshape(n, n)
            G = torch.matmul(T[flip], T.t()).reshape(n, n, n, n)
            G = G - torch.eye(n, dtype=torch.float64).cuda()[None, :, :, None] * gamma[:, None, None, :]
            return {"gamma": gamma, "Gamma": G}
        left = T[flip]
        d = torch.from_numpy(x["d"]).cuda()
        out = torch.empty((n * n, n * n, n * n), dtype=torch.float64).cuda()
        for y in range(n * n):
            out[:, :, y] = torch.matmul(left, ci.all(ci.excite(y, d)).t())
        return {"rdm3": out.reshape((n,) * 6)}
    fock = _Fock(n, case["na"], case["nb"])
    if op == "sigma":
        k, b = case["k"], x["bonds"]
        L, R = _products(b, x["sites"], 0, k)[0], _products(b, x["sites"], k + 2, n)[:, :, 0]
        t, where = _dense(b[k], b[k + 2], 2, x["psi"])
        t = torch.from_numpy(t).cuda()
        full = torch.matmul(torch.matmul(L, t.reshape(t.shape[0], -1)).reshape(-1, t.shape[2]), R).reshape(-1)
        hc = torch.zeros_like(full)
        hc[fock.index] = fock.apply_h(x["h"], x["B"], full[fock.index])
        back = torch.matmul(L.t().contiguous(), hc.reshape(L.shape[0], -1)).reshape(-1, R.shape[1])
        return {"sigma": torch.matmul(back, R.t().contiguous()).reshape(-1)[torch.from_numpy(where).cuda()]}
    c = _products(x["bonds"], x["sites"], 0, n).reshape(-1)[fock.index]
    c = c / c.norm()
    T = fock.all(c)
    flip = torch.arange(n * n).reshape(n, n).t().reshape(-1).cuda()
    gamma = torch.matmul(T, c).reshape(n, n)
    G = torch.matmul(T[flip], T.t()).reshape(n, n, n, n)
    G = G - torch.eye(n, dtype=torch.float64).cuda()[None, :, :, None] * gamma[:, None, None, :]
    F = torch.from_numpy(x["B"]).cuda().reshape(-1, n * n)
    # B_pq and B_rs enter (pq|rs) alike
    G = G.reshape(n * n, n * n)
    dB = 0.5 * (torch.matmul(F, G) + torch.matmul(F, G.t().contiguous()))
    e = float((gamma * torch.from_numpy(x["h"]).cuda()).sum() + 0.5 * (F * dB).sum())
    return {"energy": np.array([e]), "dh": gamma, "dB": dB.reshape(-1, n, n)}
