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
