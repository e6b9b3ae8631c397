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


@pytest.mark.parametrize("norb,na,nb,nd", [(9, 4, 3, 3), (12, 4, 4, 200), (12, 4, 4, 1100), (36, 3, 2, 300)])
def test_repeated_determinants_against_the_dense_double_loop(norb, na, nb, nd):
    """One determinant three times and another twice, next to each other and far
    apart: rows, product and energy as the dense double loop has them."""
    import asci_synth as syn
    import oracle
    import paper_2303_05688_amd as asci
    from gpu_util import host, to_dev

    c = syn.make_case(norb, na, nb, nd, seed=norb + nd, sampler="level", tau=max(nd / 10.0, 1.0))
    dets = np.concatenate([c["dets"], c["dets"][[0, nd - 1, 0]]])
    dets = np.ascontiguousarray(np.insert(dets, 1, c["dets"][1], axis=0))  # rows 1 and 2
    m = len(dets)
    c["dets"], c["coeffs"] = dets, np.random.default_rng(nd).normal(size=m)
    d = to_dev(c)
    H = asci.HMat(d["h"], d["eri"], norb, na, nb, d["dets"], ecore=0.7)
    rp, cols, vals = (host(t) for t in H.export())
    want, wabs = oracle.hamiltonian(c["h"], c["eri"], dets, ecore=0.7, with_abs=True)
    rows = np.repeat(np.arange(m), np.diff(rp))
    a, b = dets[:, 0], dets[:, 1]
    pop = np.vectorize(lambda x: bin(int(x)).count("1"), otypes=[int])
    diff = pop(a[:, None] ^ a[None, :]) + pop(b[:, None] ^ b[None, :])
    assert len(cols) == (diff <= 4).sum() and (diff[rows, cols] <= 4).all()
    w = want[rows, cols]
    assert (np.abs(vals - w) <= np.maximum(1e-12 * np.abs(w), 64 * U * wabs[rows, cols])).all()
    got = np.zeros((m, m))
    got[rows, cols] = vals
    for i, j in ((1, 2), (0, m - 1), (0, m - 3), (m - 2, nd)):
        assert (dets[i] == dets[j]).all() and got[i, j] == got[i, i] == got[j, i]
    x = np.abs(c["coeffs"])
    y = host(H.matvec(d["coeffs"]))
    assert (np.abs(y - want @ c["coeffs"]) <= (64 + 2 * m) * U * (wabs @ x)).all()
    e = asci.energy(d["h"], d["eri"], norb, na, nb, d["dets"], d["coeffs"], ecore=0.7)
    assert abs(e - c["coeffs"] @ want @ c["coeffs"]) <= (64 + 2 * m) * U * (x @ wabs @ x)


def test_a_repeated_start_determinant_is_refused_by_the_loop():
    import asci_synth as syn
    import paper_2303_05688_amd as asci
    from gpu_util import to_dev

    c = syn.make_case(9, 4, 3, 4, seed=2, sampler="level", tau=2.0)
    c["dets"] = np.ascontiguousarray(c["dets"][[0, 1, 1, 3]])
    d = to_dev(c)
    with pytest.raises(asci.AsciError) as err:
        asci.run(d["h"], d["eri"], 9, 4, 3, d["dets"], d["coeffs"], asci.loop_options(20, max_iter=2))
    assert err.value.code == asci.ASCI_EINVAL and "duplicate" in str(err.value)
