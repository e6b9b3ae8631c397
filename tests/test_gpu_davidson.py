"""The Davidson kernels at the edges of their blocks (256 rows, four columns a
workgroup, 512 workgroups striding over more than 131072 rows) and of the
subspace, against numpy's dense eigensolver or the residual of an independent
product.  An eigenvalue from a residual r and a gap g is off by at most r^2/g."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _hmat(n, na, ndets, seed):
    import asci_synth as syn
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    rng = np.random.default_rng(seed)
    h, eri = syn.integrals(n, rng)
    dets = np.array(syn.level_dets(n, na, na, ndets, rng), dtype=np.uint64)
    d = gu.to_dev({"h": h, "eri": eri, "dets": dets, "coeffs": np.ones(ndets)})
    return asci.HMat(d["h"], d["eri"], n, na, na, d["dets"])


def _sparse(H):
    import gpu_util as gu
    import scipy.sparse as sp

    rp, cols, vals = (gu.host(t) for t in H.export())
    return sp.csr_matrix((vals, cols, rp), shape=(H.nrows, H.nrows))


@pytest.mark.parametrize("subspace", [2, 3, 4, 5, 8, 9, 24, 48])
@pytest.mark.parametrize("ndets", [1, 2, 3, 255, 256, 257, 513])
def test_davidson_edges(ndets, subspace):
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    H = _hmat(9, 4, ndets, 50 + ndets)
    w, _ = np.linalg.eigh(_sparse(H).toarray())
    gap = w[1] - w[0] if ndets > 1 else 1.0
    e, vec, res, it = asci.davidson(H, max_subspace=subspace, max_iter=3000, tol=1e-7)
    v = gu.host(vec)
    assert res <= 1e-7 and gap > 1e-3
    assert abs(e - w[0]) <= 1e-14 / gap + 1e-11 * max(abs(w[0]), 1.0)
    assert abs(np.linalg.norm(v) - 1.0) <= 1e-12
    assert np.linalg.norm(_sparse(H) @ v - e * v) <= 2e-7
    H.close()


@pytest.mark.parametrize("ndets", [131072, 131073, 140001])
def test_davidson_many_rows(ndets):
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    H = _hmat(20, 8, ndets, 7)
    e, vec, res, it = asci.davidson(H, max_subspace=10, max_iter=1000, tol=1e-7)
    M, v = _sparse(H), gu.host(vec)
    assert res <= 1e-7 and abs(np.linalg.norm(v) - 1.0) <= 1e-12
    assert np.linalg.norm(M @ v - e * v) <= 2e-7
    assert e < M.diagonal().min()
    H.close()


def _jacobi_lowest(A):
    """Lowest eigenvector by cyclic Jacobi rotations, with the sign they give it."""
    A, m = A.copy(), len(A)
    Q = np.eye(m)
    for _ in range(60):
        if (A ** 2).sum() - (np.diag(A) ** 2).sum() <= 1e-28 * (A ** 2).sum():
            break
        for p in range(m - 1):
            for q in range(p + 1, m):
                if A[p, q] == 0.0:
                    continue
                tau = (A[q, q] - A[p, p]) / (2.0 * A[p, q])
                t = (1.0 if tau >= 0 else -1.0) / (abs(tau) + np.sqrt(1.0 + tau * tau))
                c = 1.0 / np.sqrt(1.0 + t * t)
                R = np.array([[c, t * c], [-t * c, c]])
                A[:, [p, q]] = A[:, [p, q]] @ R
                A[[p, q]] = R.T @ A[[p, q]]
                Q[:, [p, q]] = Q[:, [p, q]] @ R
    k = int(np.argmin(np.diag(A)))
    return A[k, k], Q[:, k]


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("subspace", [4, 12])
def test_davidson_sign(subspace, seed):
    """The eigenvector's sign is that of the same iteration with the projected
    problem solved by Jacobi rotations."""
    import gpu_util as gu
    import paper_2303_05688_amd as asci
    import torch

    H = _hmat(9, 4, 120, 900 + seed)
    M = _sparse(H).toarray()
    D = np.diag(M)
    g = np.random.default_rng(seed).normal(size=120)
    V = [g / np.linalg.norm(g)]
    W = [M @ V[0]]
    for _ in range(400):
        theta, c = _jacobi_lowest(np.array([[a @ b for b in W] for a in V]))
        u = sum(x * y for x, y in zip(c, V))
        r = sum(x * y for x, y in zip(c, W)) - theta * u
        if np.linalg.norm(r) <= 1e-7:
            break
        t = r / (D - theta)
        if len(V) == subspace:
            V, W = [u], [M @ u]
        for _ in range(2):
            for x in V:
                t = t - (x @ t) * x
        V.append(t / np.linalg.norm(t))
        W.append(M @ V[-1])
    e, vec, res, it = asci.davidson(H, guess=torch.from_numpy(g).to("cuda:0"), max_subspace=subspace, max_iter=400, tol=1e-7)
    w = np.linalg.eigvalsh(M)
    # two vectors of residual 1e-7 each
    assert np.linalg.norm(gu.host(vec) - u) <= 4e-7 / (w[1] - w[0])
    H.close()


@pytest.mark.parametrize("ndets", [300, 5000])
def test_davidson_products(ndets):
    """A converged guess takes one product with H and returns that vector; a
    solve takes at most one more than its iterations."""
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    H = _hmat(16, 6, ndets, 77)
    e0, v0, _, it0 = asci.davidson(H, max_subspace=12, max_iter=400, tol=1e-9)

    def solve(**kw):
        H.ctx.set_profiling(True)
        r = asci.davidson(H, max_subspace=12, max_iter=400, **kw)
        n = H.ctx.profile()["spmv"][1]
        H.ctx.set_profiling(False)
        return r, n

    (e, vec, res, it), n = solve(guess=v0, tol=1e-6)
    assert (it, n) == (1, 1) and res <= 1e-6
    assert abs(e - e0) <= 1e-11 * max(abs(e0), 1.0)
    a, b = gu.host(vec), gu.host(v0)
    assert min(np.linalg.norm(a - b), np.linalg.norm(a + b)) <= 1e-12
    (e, vec, res, it), n = solve(tol=1e-9)
    assert it == it0 > 3 and n <= it + 1 and res <= 1e-9 and e == e0
    H.close()
