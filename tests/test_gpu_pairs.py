"""The determinant-pair sweep (H over a set, the variational energy) at the
sizes where it can go wrong: one determinant, the edges of a column tile (1024)
and of a workgroup's rows, and the set sizes where the rows per wavefront change
(65,536 and 131,072, sampled rows)."""
import numpy as np
import pytest

U = 2.0 ** -53
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norb,na,nb,nd", [(9, 4, 3, 1), (9, 4, 3, 2), (9, 4, 3, 9), (12, 4, 4, 1023), (12, 4, 4, 1024),
                                           (12, 4, 4, 1025), (36, 3, 2, 1025), (12, 5, 3, 2100)])
def test_small_sets_against_the_dense_double_loop(norb, na, nb, nd):
    import asci_synth as syn
    import oracle
    import paper_2303_05688_amd as asci
    from gpu_util import host, to_dev

    c = syn.make_case(norb, na, nb, nd, seed=norb + nd, sampler="level", tau=max(nd / 10.0, 1.0))
    d = to_dev(c)
    H = asci.HMat(d["h"], d["eri"], norb, na, nb, d["dets"], ecore=0.7)
    rp, cols, vals = (host(t) for t in H.export())
    want, wabs = oracle.hamiltonian(c["h"], c["eri"], c["dets"], ecore=0.7, with_abs=True)
    rows = np.repeat(np.arange(nd), np.diff(rp))
    assert (np.diff(rows * nd + cols) > 0).all()
    a, b = c["dets"][:, 0], c["dets"][:, 1]
    pop = np.vectorize(lambda x: bin(int(x)).count("1"), otypes=[int])
    diff = pop(a[:, None] ^ a[None, :]) + pop(b[:, None] ^ b[None, :]) if nd <= 1025 else None
    if diff is not None:
        assert len(cols) == (diff <= 4).sum() and (diff[rows, cols] <= 4).all()
    else:
        assert (want[rows, cols] != 0).sum() == (want != 0).sum()
    w = want[rows, cols]
    assert (np.abs(vals - w) <= np.maximum(1e-12 * np.abs(w), 64 * U * wabs[rows, cols])).all()
    # every term of the quadratic form carries its element's rounding, and the
    # sum of nd^2 of them at most that many more
    e = asci.energy(d["h"], d["eri"], norb, na, nb, d["dets"], d["coeffs"], ecore=0.7)
    x = np.abs(c["coeffs"])
    assert abs(e - c["coeffs"] @ want @ c["coeffs"]) <= (64 + 2 * nd) * U * (x @ wabs @ x)


@pytest.mark.parametrize("nd", [65535, 65536, 131072])
def test_large_sets_by_sampled_rows(nd):
    import asci_synth as syn
    import oracle
    import paper_2303_05688_amd as asci
    from gpu_util import host, to_dev

    norb, na, nb = 24, 5, 5
    c = syn.make_case(norb, na, nb, nd, seed=nd, sampler="level", tau=nd / 10.0)
    d = to_dev(c)
    H = asci.HMat(d["h"], d["eri"], norb, na, nb, d["dets"])
    rp, cols, vals = (host(t) for t in H.export())
    a, b = c["dets"][:, 0], c["dets"][:, 1]
    table = np.array([bin(i).count("1") for i in range(1 << 12)], dtype=np.int64)
    pop = lambda v: table[(v & np.uint64(0xFFF)).astype(np.int64)] + table[(v >> np.uint64(12)).astype(np.int64)]  # noqa: E731
    rng = np.random.default_rng(nd)
    for i in [0, 1, nd - 1, *rng.integers(0, nd, 30)]:
        want = np.nonzero(pop(a ^ a[i]) + pop(b ^ b[i]) <= 4)[0]
        got = cols[rp[i]:rp[i + 1]]
        assert len(got) == len(want) and (got == want).all()
        for k in rng.integers(0, len(want), 5):
            v = oracle.helem(c["h"], c["eri"], c["dets"][i], c["dets"][want[k]])
            assert abs(vals[rp[i] + k] - v) <= 1e-11 * max(1.0, abs(v))
    # the energy takes every pair once, the rows' dot products twice
    hc = host(H.matvec(d["coeffs"]))
    e = asci.energy(d["h"], d["eri"], norb, na, nb, d["dets"], d["coeffs"])
    assert abs(e - c["coeffs"] @ hc) <= 1e-11 * (np.abs(c["coeffs"]) @ np.abs(hc))
