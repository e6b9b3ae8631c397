"""Sorts on both sides of the line between merged and digit-by-digit ones
(1,572,864 records): the final order of a search with a large k, synchronous and
asynchronous, and the core set of a large determinant set, ties included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LINE = 3 << 19


def test_final_order_of_a_large_selection():
    import asci_synth as syn
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    n, na, nb, nd = 20, 8, 8, 400
    rng = np.random.default_rng(3)
    h, eri = syn.integrals(n, rng)
    dets = np.array(syn.uniform_dets(n, na, nb, nd, rng), dtype=np.uint64)
    # few distinct factors: many tied scores
    h, eri = np.round(h / 0.125) * 0.125, np.round(eri / 0.125) * 0.125
    d = gu.to_dev({"h": h, "eri": eri, "dets": dets, "coeffs": np.sign(rng.normal(size=nd)) * 0.0625})
    where = (d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], -100.25)
    k, _, sc = (gu.host(x) for x in asci.candidates(*where))
    order = np.lexsort((k[:, 1], k[:, 0], ~gu.abs_bits(sc)))
    k, sc = k[order], sc[order]
    assert len(sc) > LINE + 4097 and len(np.unique(gu.abs_bits(sc))) < len(sc) // 2
    for take in (LINE, LINE + 1, LINE + 4097, len(sc), len(sc) + 5):
        m = min(take, len(sc))
        gk, gs = (gu.host(x) for x in asci.search(*where, take))
        assert len(gs) == m
        assert (gk == k[:m]).all() and (gs.view(np.uint64) == sc[:m].view(np.uint64)).all(), take
        r = asci.SearchRequest(*where, take)
        count, status, flags = asci.async_status(asci.search_async(r))
        assert (count, status, flags) == (m, 0, 0)
        gk, gs = (gu.host(x) for x in r.result(count))
        assert (gk == k[:m]).all() and (gs.view(np.uint64) == sc[:m].view(np.uint64)).all(), take


@pytest.mark.parametrize("nd,ncore", [(LINE, 1000), (LINE + 1, 1000), (LINE + 4097, LINE + 1), (2_000_003, 1)])
def test_core_set_of_a_large_determinant_set(nd, ncore):
    import torch

    import paper_2303_05688_amd as asci

    n, ne = 24, 4
    rng = np.random.default_rng(nd)
    occ = np.argsort(rng.random((2, 4096, n)), axis=2)[:, :, :ne].astype(np.uint64)
    s = np.unique(np.bitwise_or.reduce(np.uint64(1) << occ, axis=2).ravel())
    pick = rng.permutation(len(s) ** 2)[:nd]  # distinct (alpha, beta) pairs
    dets = np.ascontiguousarray(np.stack([s[pick // len(s)], s[pick % len(s)]], 1))
    c = rng.choice([1.0, -1.0, 0.5, -0.25, 2.0 ** -900], size=nd)
    core = np.sort(np.lexsort((np.arange(nd), -np.abs(c)))[:ncore])
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")  # noqa: E731
    got = asci.class_counts(n, ne, ne, up(dets.view(np.int64)).view(torch.uint64), up(c), ncore=ncore, constraint_level=4)
    want = asci.class_counts(n, ne, ne, up(dets[core].view(np.int64)).view(torch.uint64), up(c[core]), constraint_level=4)
    assert (got[0] == want[0]).all() and (got[1] == want[1]).all()
