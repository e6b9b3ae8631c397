"""Final segments of the sort-and-accumulate at the sizes where they can go
wrong: a target with as many contributions as one wavefront's share of records
(finish_cap / 8), one less, one more and several times as many, for every finish
capacity; candidates against the oracle, N_a bit-identical whatever the
capacity (the summation order does not depend on it)."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _connected(n, na, nb):
    """The singles and doubles of the aufbau determinant, without it: each
    contributes once to the aufbau target."""
    a0, b0 = (1 << na) - 1, (1 << nb) - 1

    def moves(s, ne, k):
        for holes in itertools.combinations(range(ne), k):
            for parts in itertools.combinations(range(ne, n), k):
                t = s
                for p in holes:
                    t &= ~(1 << p)
                for p in parts:
                    t |= 1 << p
                yield t

    out = [(a, b0) for k in (1, 2) for a in moves(a0, na, k)]
    out += [(a0, b) for k in (1, 2) for b in moves(b0, nb, k)]
    out += [(a, b) for a in moves(a0, na, 1) for b in moves(b0, nb, 1)]
    return np.array(out, dtype=np.uint64)


@pytest.mark.parametrize("norb", [10, 34])
@pytest.mark.parametrize("ndets", [127, 128, 129, 257, 511, 512, 513, 800])
def test_heavy_target_by_finish_capacity(norb, ndets):
    import asci_synth as syn
    import gpu_util as gu
    import oracle
    import paper_2303_05688_amd as asci

    # 34 orbitals (two-word keys) with few electrons keep the oracle quick
    na, nb = (4, 4) if norb == 10 else (2, 2)
    rng = np.random.default_rng(1000 * norb + ndets)
    h, eri = syn.integrals(norb, rng)
    dets = _connected(norb, na, nb)
    dets = np.ascontiguousarray(dets[np.sort(rng.permutation(len(dets))[:ndets])])
    case = {"h": h, "eri": eri, "dets": dets, "coeffs": syn.coefficients(ndets, ndets, rng)}
    E0 = oracle.energy(h, eri, dets, case["coeffs"])
    want = oracle.search_all(h, eri, norb, na, nb, dets, case["coeffs"], E0)
    d = gu.to_dev(case)
    first = None
    for cap in (4096, 2048, 1024):
        ctx = asci.Context(0)
        ctx.set_param("finish_cap", cap)
        k, num, sc = (gu.host(x) for x in asci.candidates(d["h"], d["eri"], norb, na, nb, d["dets"], d["coeffs"], E0, ctx=ctx))
        gu.assert_candidates(k, num, sc, want)
        if first is None:
            first = (num, sc)
        assert (num.view(np.uint64) == first[0].view(np.uint64)).all()
        assert (sc.view(np.uint64) == first[1].view(np.uint64)).all()
        # several class batches: the k-th score of the earlier ones prunes the later
        full = asci.search(d["h"], d["eri"], norb, na, nb, d["dets"], d["coeffs"], E0, 50, ctx=ctx)
        part = asci.search(d["h"], d["eri"], norb, na, nb, d["dets"], d["coeffs"], E0, 50, ctx=ctx, pair_buffer_bytes=32 * 40000)
        assert ctx.get_param("last_batches") > 1
        assert (gu.host(full[0]) == gu.host(part[0])).all()
        assert (gu.host(full[1]) == gu.host(part[1])).all()
        ctx.close()


@pytest.mark.parametrize("norb", [12, 34])
def test_smallest_finish_capacity_takes_the_shares_of_the_next(norb):
    """A wavefront's share is 256 records at least: finish_cap 1024 divides as
    2048 does, and finer than 4096."""
    import asci_synth as syn
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    ne = 4 if norb == 12 else 2
    c = syn.make_case(norb, ne, ne, 300, seed=norb, sampler="level", tau=30.0)
    d = gu.to_dev(c)
    finals, out = [], []
    for cap in (4096, 2048, 1024):
        ctx = asci.Context(0)
        ctx.set_param("finish_cap", cap)
        out.append([gu.host(x) for x in asci.search(d["h"], d["eri"], norb, ne, ne, d["dets"], d["coeffs"], -3.5, 500, ctx=ctx)])
        finals.append(ctx.get_param("last_finals"))
        ctx.close()
    assert finals[0] < finals[1] == finals[2]
    for k, sc in out[1:]:
        assert (k == out[0][0]).all() and (sc.view(np.uint64) == out[0][1].view(np.uint64)).all()
