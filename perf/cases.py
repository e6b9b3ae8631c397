"""Timed cases of the ASCI determinant search: what a program that uses this
library has it do, through the public entry points of paper_2303_05688_amd.

A case is a dict of plain values.  "kind" names the entry point:

  search      asci.search: the k best new determinants (one call per iteration
              of an ASCI run, and the request of a serving program)
  batch       asci.search_batch: many small searches in one call
  candidates  asci.candidates: every new determinant with N_a and A_a
  pt2         asci.pt2: the second-order energy that closes a run
  energy      asci.energy: <C|H|C>, the E_0 that a search needs
  hmat        asci.HMat: H over the determinant set, exported, and one H x
  loop        asci.run: the whole ASCI loop from the Hartree-Fock determinant
              (search, selection, H, Davidson, PT2)

Inputs follow the recipe of the repository's synthetic workloads (integrals
that decay with orbital distance, determinants drawn by excitation level from
the aufbau one, coefficients that decay with the index).  E_0 is a
variational energy's stand-in: below the lowest diagonal element of the input
set by a correlation energy, as in a converged iteration.
"""
import math

import numpy as np
import torch

import paper_2303_05688_amd as asci

CORRELATION = 0.25  # E_0 lies this far below the lowest diagonal element


def comb(n, k):
    return math.comb(n, k) if 0 <= k <= n else 0


def pairs_per_det(n, na, nb):
    va, vb = n - na, n - nb
    return na * va + nb * vb + comb(na, 2) * comb(va, 2) + comb(nb, 2) * comb(vb, 2) + na * va * nb * vb


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the repository's smallest workload: a few hundred determinants, where launches and round trips are the time
        dict(name="search 8e12o", kind="search", norb=12, nalpha=4, nbeta=4, ndets=201, ncore=0, k=2000),
        # a small request of a batch or a serving mix (10 to 20 orbitals, 10^2 to 10^3 cores), odd orbital count
        dict(name="search 10e17o", kind="search", norb=17, nalpha=5, nbeta=5, ndets=613, ncore=0, k=6130),
        # the repository's middle workload, one class batch
        dict(name="search 16e20o", kind="search", norb=20, nalpha=8, nbeta=8, ndets=10000, ncore=0, k=100000),
        # the headline: the Cr2 shape, 6.7e9 pairs in several class batches
        dict(name="search 24e30o", kind="search", norb=30, nalpha=12, nbeta=12, ndets=100000, ncore=0, k=1000000),
        # two-word keys (more than 32 orbitals)
        dict(name="search 20e36o", kind="search", norb=36, nalpha=10, nbeta=10, ndets=2000, ncore=0, k=20000),
        # an open-shell iteration with fewer core determinants than determinants (N_cdets < N_tdets), ragged sizes
        dict(name="search 8a5b23o core", kind="search", norb=23, nalpha=8, nbeta=5, ndets=20011, ncore=3001, k=20011),
        # every candidate with its numerator, for analysis and selection outside the library
        dict(name="candidates 12e18o", kind="candidates", norb=18, nalpha=6, nbeta=6, ndets=2000),
        # the perturbative correction over the same candidates
        dict(name="pt2 16e20o", kind="pt2", norb=20, nalpha=8, nbeta=8, ndets=5000),
        # the variational energy of a wave function before its first search
        dict(name="energy 16e20o", kind="energy", norb=20, nalpha=8, nbeta=8, ndets=10000),
        # the Hamiltonian of the variational step
        dict(name="hmat 16e20o", kind="hmat", norb=20, nalpha=8, nbeta=8, ndets=20000),
        # many small searches at once (scans over geometries or fragments)
        dict(name="batch of 24 small", kind="batch", count=24, norb_lo=10, norb_hi=20, ndets_lo=100, ndets_hi=1000),
        # the whole method, open shell
        dict(name="loop 8a6b19o", kind="loop", norb=19, nalpha=8, nbeta=6, ntdets=5000, ncore=2000, iters=3),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _shape(rng, n_lo, n_hi, e_hi):
    """norb and the electrons of each spin: closed or open shell."""
    n = rng.randint(n_lo, n_hi)
    na = rng.randint(2, min(e_hi, n - 2))
    nb = max(1, na - rng.choice([0, 0, 0, 1, 2, 3]))
    return n, na, nb


def _ndets(rng, n, na, nb, lo, hi, most_pairs):
    nd = int(round(_log_uniform(rng, lo, hi)))
    nd = min(nd, max(1, comb(n, na) * comb(n, nb) // 4), max(1, int(most_pairs // pairs_per_det(n, na, nb))))
    return max(1, nd)


def draw(rng):
    kind = rng.choice(["search"] * 5 + ["candidates", "pt2", "energy", "hmat", "batch", "loop"])
    if kind == "search":
        n, na, nb = _shape(rng, 10, 40, 14)
        nd = _ndets(rng, n, na, nb, 1e2, 1e5, 3e9)
        ncore = rng.choice([0, 0, max(1, int(nd * rng.uniform(0.05, 0.9)))])
        return dict(kind=kind, norb=n, nalpha=na, nbeta=nb, ndets=nd, ncore=ncore, k=max(1, int((ncore or nd) * rng.uniform(1, 12))))
    if kind == "candidates":
        n, na, nb = _shape(rng, 10, 24, 9)
        return dict(kind=kind, norb=n, nalpha=na, nbeta=nb, ndets=_ndets(rng, n, na, nb, 1e2, 1e4, 6e7))
    if kind == "pt2":
        n, na, nb = _shape(rng, 12, 36, 12)
        return dict(kind=kind, norb=n, nalpha=na, nbeta=nb, ndets=_ndets(rng, n, na, nb, 1e2, 5e4, 1e9))
    if kind in ("energy", "hmat"):
        n, na, nb = _shape(rng, 12, 36, 12)
        return dict(kind=kind, norb=n, nalpha=na, nbeta=nb, ndets=_ndets(rng, n, na, nb, 3e2, 3e4, 1e15))
    if kind == "batch":
        lo = rng.randint(10, 16)
        return dict(kind=kind, count=rng.randint(5, 30), norb_lo=lo, norb_hi=rng.randint(lo, 20), ndets_lo=100, ndets_hi=rng.randint(300, 1000))
    n = rng.randint(14, 22)
    na = rng.randint(5, 9)
    nt = int(round(_log_uniform(rng, 1e3, 1e4)))
    return dict(kind=kind, norb=n, nalpha=na, nbeta=na - rng.randint(1, 3), ntdets=nt, ncore=max(1, int(nt * rng.uniform(0.2, 1))), iters=3)


def work(case):
    """What one pass cannot do without: every input read once, every output
    written once; one product and one sum for each contribution H_ai C_i (for
    energy and hmat: for the couplings inside the set, some hundreds a row)."""
    kind = case["kind"]
    if kind == "batch":
        parts = [work(c) for c in _batch(case, 0)]
        return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}
    n, na, nb = case["norb"], case["nalpha"], case["nbeta"]
    nd = case.get("ndets") or case["ntdets"]
    per = pairs_per_det(n, na, nb)
    pairs = (case.get("ncore") or nd) * per
    read = 8 * n ** 4 + 8 * n ** 2 + 24 * nd
    if kind == "search":
        return {"bytes": read + 24 * min(case["k"], pairs), "flops": 2 * pairs}
    if kind == "candidates":
        return {"bytes": read + 32 * (pairs // 3), "flops": 2 * pairs}
    if kind == "pt2":
        return {"bytes": read + 16, "flops": 2 * pairs}
    couplings = nd * min(nd, 400)
    if kind == "energy":
        return {"bytes": read + 8, "flops": 2 * couplings}
    if kind == "hmat":
        return {"bytes": read + 12 * couplings + 24 * nd, "flops": 2 * couplings}
    return {"bytes": read + 12 * couplings, "flops": 2 * case["iters"] * pairs}


# ---------------------------------------------------------------- inputs
def _integrals(n, rng):
    """h (n x n) and (pq|rs) (n^4): decaying with orbital distance, 8-fold symmetric bit for bit."""
    base = np.repeat([-2.0, 0.0, 2.0], [n // 3 + (b < n % 3) for b in range(3)])
    h = np.diag(np.sort(np.clip(base + rng.uniform(-0.1, 0.1, n), -3.0, 3.0)))
    iu = np.triu_indices(n, 1)
    h[iu] = rng.normal(0.0, 0.3, len(iu[0])) * np.exp(-(iu[1] - iu[0]) / 4.0)
    h.T[iu] = h[iu]
    p, q = np.tril_indices(n)
    i, j = np.tril_indices(len(p))
    p, q, r, s = p[i], q[i], p[j], q[j]
    v = 0.1 * np.exp(-(p - q + r - s) / 3.0) * rng.normal(0.0, 1.0, len(i)) + 0.5 * ((p == q) & (r == s))
    eri = np.zeros((n, n, n, n))
    for a, b, c, d in ((p, q, r, s), (q, p, r, s), (p, q, s, r), (q, p, s, r)):
        eri[a, b, c, d] = v
        eri[c, d, a, b] = v
    return h, eri


def _subsets(rng, rows, width, size):
    """For each row, a uniform subset of `size[row]` of `width` places, as booleans."""
    if width == 0:
        return np.zeros((rows, 0), bool)
    rank = np.argsort(np.argsort(rng.random((rows, width)), axis=1), axis=1)
    return rank < size[:, None]


def _dets(n, na, nb, count, rng):
    """`count` distinct determinants: aufbau first, then by excitation level L with P(L) ~ exp(-L)."""
    va, vb = n - na, n - nb
    lmax = min(na, va) + min(nb, vb)
    bit = np.uint64(1) << np.arange(n, dtype=np.uint64)
    fa, fb = np.uint64((1 << na) - 1), np.uint64((1 << nb) - 1)
    levels = np.arange(1, lmax + 1)
    pl = np.exp(-levels.astype(float))
    pl /= pl.sum()
    cdf = np.ones((lmax + 1, lmax + 1))
    for L in levels:
        w = np.array([float(comb(na, x) * comb(va, x) * comb(nb, L - x) * comb(vb, L - x)) for x in range(lmax + 1)])
        cdf[L] = np.cumsum(w / w.sum())
    got = np.array([[fa, fb, 0]], dtype=np.uint64)
    rounds = 0
    while len(got) < count:
        rows = max(1024, 2 * (count - len(got)))
        # a set that nearly fills the low levels is completed from flatter draws
        p = pl if rounds < 12 else np.full(lmax, 1.0 / lmax)
        lev = rng.choice(levels, size=rows, p=p)
        la = np.minimum((rng.random(rows)[:, None] > cdf[lev]).sum(1), lev)
        lb = lev - la
        ha, pa = _subsets(rng, rows, na, la), _subsets(rng, rows, va, la)
        hb, pb = _subsets(rng, rows, nb, lb), _subsets(rng, rows, vb, lb)
        word = lambda m, b: (m * b).sum(1, dtype=np.uint64)  # noqa: E731
        a = (fa & ~word(ha, bit[:na])) | word(pa, bit[na:])
        b = (fb & ~word(hb, bit[:nb])) | word(pb, bit[nb:])
        got = np.concatenate([got, np.stack([a, b, lev.astype(np.uint64)], 1)])
        order = np.lexsort((np.arange(len(got)), got[:, 1], got[:, 0]))
        first = np.ones(len(got), bool)
        first[1:] = (got[order[1:], :2] != got[order[:-1], :2]).any(1)
        got = got[np.sort(order[first])]
        rounds += 1
    got = got[:count]
    return np.ascontiguousarray(got[np.argsort(got[:, 2], kind="stable"), :2])


def _occupations(s, n):
    return ((s[:, None] >> np.arange(n, dtype=np.uint64)) & np.uint64(1)).astype(np.float64)


def _diagonal(h, eri, oa, ob):
    """H_aa of occupation rows (numpy arrays or torch tensors alike)."""
    e = (lambda s, x: torch.einsum(s, x)) if isinstance(eri, torch.Tensor) else np.einsum
    J = e("ppqq->pq", eri)
    X = J - e("pqqp->pq", eri)
    hd = e("pp->p", h)
    return oa @ hd + ob @ hd + 0.5 * ((oa @ X) * oa).sum(1) + 0.5 * ((ob @ X) * ob).sum(1) + ((oa @ J) * ob).sum(1)


def _host_inputs(case, seed):
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, case["norb"]])
    n, na, nb, nd = case["norb"], case["nalpha"], case["nbeta"], case["ndets"]
    h, eri = _integrals(n, rng)
    # where the outputs' sizes follow from the determinants, these come from the case alone
    fixed = case["kind"] in ("candidates", "hmat")
    dets = _dets(n, na, nb, nd, np.random.default_rng([n, na, nb, nd]) if fixed else rng)
    c = rng.normal(0.0, 1.0, nd) * np.exp(-np.arange(nd) / max(nd / 10.0, 1.0))
    c /= np.linalg.norm(c)
    e0 = float(_diagonal(h, eri, _occupations(dets[:, 0], n), _occupations(dets[:, 1], n)).min()) - CORRELATION
    return h, eri, dets, c, e0


def _to_gpu(case, seed):
    h, eri, dets, c, e0 = _host_inputs(case, seed)
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    return dict(case=case, h=up(h), eri=up(eri), dets=up(dets.view(np.int64)).view(torch.uint64), c=up(c), e0=e0)


def _batch(case, seed):
    """The small searches of a batch: sizes from the case alone, so that every seed has the same work."""
    rng = np.random.default_rng([case["count"], case["norb_lo"], case["norb_hi"], case["ndets_hi"]])
    out = []
    for _ in range(case["count"]):
        n = int(rng.integers(case["norb_lo"], case["norb_hi"] + 1))
        na = min(int(rng.integers(2, 7)), n - 2)
        nd = int(round(10 ** rng.uniform(math.log10(case["ndets_lo"]), math.log10(case["ndets_hi"]))))
        nd = max(1, min(nd, comb(n, na) ** 2 // 4))
        out.append(dict(kind="search", norb=n, nalpha=na, nbeta=na, ndets=nd, ncore=0, k=10 * nd))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        reqs = []
        for i, c in enumerate(_batch(case, seed)):
            s = _to_gpu(c, seed + 1000 * i)
            reqs.append(asci.SearchRequest(s["h"], s["eri"], c["norb"], c["nalpha"], c["nbeta"], s["dets"], s["c"], s["e0"], c["k"]))
        return dict(case=case, reqs=reqs)
    if kind == "loop":
        n, na, nb = case["norb"], case["nalpha"], case["nbeta"]
        s = _to_gpu(dict(case, ndets=1), seed)
        s["case"] = case
        s["c"] = torch.ones(1, dtype=torch.float64, device="cuda")
        s["opts"] = asci.loop_options(ntdets=case["ntdets"], ncore=case["ncore"], max_iter=case["iters"], e_tol=0.0, davidson_tol=1e-6, pt2=True)
        return s
    s = _to_gpu(case, seed)
    if kind == "hmat":
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed))
        s["x"] = torch.randn(case["ndets"], dtype=torch.float64, device="cuda", generator=g)
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        res = asci.search_batch(state["reqs"])
        out = []
        for q, r in zip(state["reqs"], res):
            d, s = q.result(r.count)
            out.append((d.view(torch.int64), s))
        return out
    where = (state["h"], state["eri"], case["norb"], case["nalpha"], case["nbeta"], state["dets"])
    if kind == "search":
        d, s = asci.search(*where, state["c"], state["e0"], case["k"], ncore=case["ncore"])
        return d.view(torch.int64), s
    if kind == "candidates":
        d, num, s = asci.candidates(*where, state["c"], state["e0"])
        return d.view(torch.int64), num, s
    if kind == "pt2":
        return asci.pt2(*where, state["c"], state["e0"])
    if kind == "energy":
        return asci.energy(*where, state["c"])
    if kind == "hmat":
        H = asci.HMat(*where)
        rp, cols, vals = H.export()
        return rp, cols, vals, H.matvec(state["x"])
    r = asci.run(*where, state["c"], state["opts"])
    return r["dets"].view(torch.int64), r["coeffs"], r["energy"], r["pt2"]


# ---------------------------------------------------------------- 64-bit values
MOST_PAIRS = 3e8  # larger searches take too long (and too much memory) here


class _Oracle:
    """Plain torch: every excitation of a block of determinants, its target as
    a pair of combinatorial ranks in one integer, and H_ai."""

    def __init__(self, h, eri, n, na, nb, dets):
        d = torch.device("cuda")
        self.n, self.ne = n, (na, nb)
        self.h, self.eri = torch.from_numpy(h).to(d), torch.from_numpy(eri).to(d)
        self.dets = torch.from_numpy(dets.view(np.int64)).to(d)
        self.binom = torch.tensor([[comb(p, k) for p in range(n + 1)] for k in range(max(na, nb) + 2)], dtype=torch.int64, device=d)
        self.width = comb(n, nb)
        self.bits = torch.arange(n, device=d)
        e = self.eri
        jx = torch.diagonal(e, dim1=2, dim2=3)  # [q, p, r] = (qp|rr)
        kx = torch.einsum("qrrp->qpr", e)
        self.same = (jx - kx).reshape(n * n, n).T.contiguous()
        self.other = jx.reshape(n * n, n).T.contiguous()
        self.flat = e.reshape(-1)

    def occ(self, s):
        return (s[:, None] >> self.bits) & 1

    def rank(self, s):
        o = self.occ(s.reshape(-1))
        k = torch.cumsum(o, 1)
        r = (o * self.binom[k.clamp(max=self.binom.shape[0] - 1), self.bits]).sum(1)
        return r.reshape(s.shape)

    def at(self, p, q, r, s):
        n = self.n
        return self.flat[((p * n + q) * n + r) * n + s]

    def lists(self, s, ne):
        o = self.occ(s)
        order = torch.argsort(1 - o, dim=1, stable=True)
        cum = torch.zeros((len(s), self.n + 1), dtype=torch.int64, device=s.device)
        cum[:, 1:] = torch.cumsum(o, 1)
        return order[:, :ne], order[:, ne:], cum

    @staticmethod
    def between(cum, p, q):
        """occupied orbitals strictly between p and q, per row"""
        lo, hi = torch.minimum(p, q), torch.maximum(p, q)
        return torch.gather(cum, 1, hi) - torch.gather(cum, 1, lo + 1)

    def singles(self, s, ne):
        occ, vir, cum = self.lists(s, ne)
        p = occ[:, :, None].expand(-1, -1, vir.shape[1]).reshape(len(s), -1)
        q = vir[:, None, :].expand(-1, occ.shape[1], -1).reshape(len(s), -1)
        t = s[:, None] ^ (1 << p) ^ (1 << q)
        return p, q, t, 1 - 2 * (self.between(cum, p, q) & 1)

    def doubles(self, s, ne):
        occ, vir, cum = self.lists(s, ne)
        i, j = torch.triu_indices(ne, ne, 1, device=s.device)
        a, b = torch.triu_indices(self.n - ne, self.n - ne, 1, device=s.device)
        big = lambda x, m: x[:, :, None].expand(-1, -1, m).reshape(len(s), -1)  # noqa: E731
        rep = lambda x, m: x[:, None, :].expand(-1, m, -1).reshape(len(s), -1)  # noqa: E731
        p, r = big(occ[:, i], len(a)), big(occ[:, j], len(a))
        q, t = rep(vir[:, a], len(i)), rep(vir[:, b], len(i))
        lo, hi = torch.minimum(r, t), torch.maximum(r, t)
        moved = ((q > lo) & (q < hi)).long() - ((p > lo) & (p < hi)).long()
        sign = 1 - 2 * ((self.between(cum, p, q) + self.between(cum, r, t) + moved) & 1)
        v = self.at(q, p, t, r) - self.at(q, r, t, p)
        return s[:, None] ^ (1 << p) ^ (1 << r) ^ (1 << q) ^ (1 << t), v * sign

    def block(self, lo, hi):
        """(target alpha, target beta, H_ai) of determinants lo..hi, each [hi - lo, m]."""
        n = self.n
        A, B = self.dets[lo:hi, 0], self.dets[lo:hi, 1]
        oa, ob = self.occ(A).double(), self.occ(B).double()
        hq = self.h.reshape(1, -1)
        fa = hq + oa @ self.same + ob @ self.other  # [row, q * n + p]
        fb = hq + ob @ self.same + oa @ self.other
        pa, qa, ta, sa = self.singles(A, self.ne[0])
        pb, qb, tb, sb = self.singles(B, self.ne[1])
        out = [(ta, B[:, None].expand_as(ta), torch.gather(fa, 1, qa * n + pa) * sa),
               (A[:, None].expand_as(tb), tb, torch.gather(fb, 1, qb * n + pb) * sb)]
        t, v = self.doubles(A, self.ne[0])
        out.append((t, B[:, None].expand_as(t), v))
        t, v = self.doubles(B, self.ne[1])
        out.append((A[:, None].expand_as(t), t, v))
        e = self.flat[(qa * n + pa)[:, :, None] * (n * n) + (qb * n + pb)[:, None, :]]
        e = e * sa[:, :, None] * sb[:, None, :]
        m, k = ta.shape[1], tb.shape[1]
        out.append((ta[:, :, None].expand(-1, m, k).reshape(len(A), -1), tb[:, None, :].expand(-1, m, k).reshape(len(A), -1), e.reshape(len(A), -1)))
        return [torch.cat(x, 1) for x in zip(*out)]

    def key(self, a, b):
        return self.rank(a) * self.width + self.rank(b)

    def blocks(self, index):
        """row ranges of about 4 million targets"""
        step = max(1, int(4e6 // max(1, pairs_per_det(self.n, *self.ne))))
        for lo in range(0, len(index), step):
            yield index[lo:lo + step]


def _exact_search(case, seed):
    n, na, nb = case["norb"], case["nalpha"], case["nbeta"]
    nq = case.get("ncore") or case["ndets"]
    if nq * pairs_per_det(n, na, nb) > MOST_PAIRS or comb(n, na) * comb(n, nb) >= 2 ** 62:
        return None
    h, eri, dets, c, e0 = _host_inputs(case, seed)
    core = np.sort(np.lexsort((np.arange(len(c)), -np.abs(c)))[:nq])
    o = _Oracle(h, eri, n, na, nb, np.ascontiguousarray(dets[core]))
    cc = torch.from_numpy(c[core]).cuda()
    keys, vals = [], []
    for rows in o.blocks(range(nq)):
        a, b, v = o.block(rows.start, rows.stop)
        keys.append(o.key(a, b).reshape(-1))
        vals.append((v * cc[rows.start:rows.stop, None]).reshape(-1))
    keys, vals = torch.cat(keys), torch.cat(vals)
    u, inv = torch.unique(keys, return_inverse=True)
    del keys
    num = torch.zeros(len(u), dtype=torch.float64, device="cuda").index_add_(0, inv, vals)
    del inv, vals
    all_dets = torch.from_numpy(dets.view(np.int64)).cuda()
    psi = torch.sort(o.key(all_dets[:, 0], all_dets[:, 1])).values
    at = torch.searchsorted(psi, u).clamp(max=len(psi) - 1)
    new = psi[at] != u
    u, num = u[new], num[new]
    den = torch.empty_like(num)
    for lo in range(0, len(u), 1 << 21):
        k = u[lo:lo + (1 << 21)]
        den[lo:lo + (1 << 21)] = e0 - _diagonal(o.h, o.eri, _unrank(o, k // o.width, na), _unrank(o, k % o.width, nb))
    return u, num, num / den


def _unrank(o, r, ne):
    """occupation rows of combinatorial ranks"""
    out = torch.zeros((len(r), o.n), dtype=torch.float64, device="cuda")
    r = r.clone()
    for j in range(ne, 0, -1):
        p = torch.searchsorted(o.binom[j].contiguous(), r, right=True) - 1
        out[torch.arange(len(r), device="cuda"), p] = 1.0
        r -= o.binom[j][p]
    return out


def _couplings(case, seed):
    """H over the determinant set: (row, column, value) sorted by row, column."""
    n, na, nb, nd = case["norb"], case["nalpha"], case["nbeta"], case["ndets"]
    if nd * pairs_per_det(n, na, nb) > 4 * MOST_PAIRS or comb(n, na) * comb(n, nb) >= 2 ** 62:
        return None
    h, eri, dets, c, _ = _host_inputs(case, seed)
    o = _Oracle(h, eri, n, na, nb, dets)
    psi, where = torch.sort(o.key(o.dets[:, 0], o.dets[:, 1]))
    rows, cols, vals = [], [], []
    for r in o.blocks(range(nd)):
        a, b, v = o.block(r.start, r.stop)
        k = o.key(a, b)
        at = torch.searchsorted(psi, k).clamp(max=nd - 1)
        hit = psi[at] == k
        i, j = torch.nonzero(hit, as_tuple=True)
        rows.append(where[at[i, j]])
        cols.append(i + r.start)
        vals.append(v[i, j])
    diag = _diagonal(o.h, o.eri, o.occ(o.dets[:, 0]).double(), o.occ(o.dets[:, 1]).double())
    me = torch.arange(nd, device="cuda")
    rows, cols, vals = torch.cat(rows + [me]), torch.cat(cols + [me]), torch.cat(vals + [diag])
    order = torch.argsort(rows * nd + cols)
    return rows[order], cols[order], vals[order], torch.from_numpy(c).cuda()


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for i, c in enumerate(_batch(case, seed)):
            out.append(exact(c, seed + 1000 * i))
        return out
    if kind in ("search", "candidates", "pt2"):
        got = _exact_search(case, seed)
        if got is None:
            return None
        _, num, score = got
        if kind == "pt2":
            return float((num * score).sum()), None
        if kind == "candidates":
            return None, num, score  # ranks grow with the strings: the order of the keys
        order = torch.sort(score.abs(), descending=True, stable=True).indices[: case["k"]]
        return None, score[order]
    if kind in ("energy", "hmat"):
        got = _couplings(case, seed)
        if got is None:
            return None
        r, c, v, coef = got
        if kind == "energy":
            return float((v * coef[r] * coef[c]).sum())
        g = torch.Generator(device="cuda")
        g.manual_seed(int(seed))
        x = torch.randn(case["ndets"], dtype=torch.float64, device="cuda", generator=g)
        y = torch.zeros(case["ndets"], dtype=torch.float64, device="cuda").index_add_(0, r, v * x[c])
        return None, None, v, y
    return None
