"""Searches under a threshold: a pilot share of the final segments bounds the
k-th |A| before the others are finished, and with both string tables targets
are rejected by a bound on their diagonal element.  The selection must be the k
largest of every candidate, bit for bit, and the candidates counted all of
them, whatever the threshold, the bound and the tables do."""
from math import comb

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _per(n, na, nb):
    va, vb = n - na, n - nb
    return na * va + nb * vb + comb(na, 2) * comb(va, 2) + comb(nb, 2) * comb(vb, 2) + na * va * nb * vb


def _case(n, na, nb, ndets, seed, quantum=None):
    import asci_synth as syn
    import gpu_util as gu

    rng = np.random.default_rng(seed)
    h, eri = syn.integrals(n, rng)
    dets = np.array(syn.uniform_dets(n, na, nb, ndets, rng), dtype=np.uint64)
    c = syn.coefficients(ndets, ndets, rng)
    if quantum is not None:
        h, eri = np.round(h / quantum) * quantum, np.round(eri / quantum) * quantum
        c = np.sign(c + 1e-30) * 2.0 ** -np.ceil(np.log2(ndets) / 2)
    return gu.to_dev({"h": h, "eri": eri, "dets": dets, "coeffs": c})


def _check(d, n, na, nb, E0, ks, tables, **kw):
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    k, _, sc = (gu.host(x) for x in asci.candidates(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], E0))
    order = np.lexsort((k[:, 1], k[:, 0], ~gu.abs_bits(sc)))[:max(ks)]
    wk, ws = k[order], sc[order]
    for t in tables:
        ctx = asci.Context(0)
        ctx.set_param("spin_tables", t)
        for kk in ks:
            gk, gs = (gu.host(x) for x in asci.search(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], E0, kk,
                                                      ctx=ctx, **kw))
            m = min(kk, len(sc))
            assert len(gs) == m and (gk == wk[:m]).all() and (gs.view(np.uint64) == ws[:m].view(np.uint64)).all(), (t, kk)
            if ctx.get_param("last_batches") == 1:
                assert ctx.get_param("last_candidates") == len(sc)


# E0 far below every diagonal element, and among them (a bound of no use)
@pytest.mark.parametrize("E0", [-100.25, 12.0])
@pytest.mark.parametrize("n,na,nb", [(14, 7, 7), (34, 3, 3)])
def test_pilot_one_batch(n, na, nb, E0):
    d = _case(n, na, nb, (1 << 26) // _per(n, na, nb) + 1, 40 + n)
    _check(d, n, na, nb, E0, [1, 1000, 1 << 18, (1 << 18) + 1], (1, 0))


def test_pilot_tied_scores():
    d = _case(14, 7, 7, (1 << 26) // _per(14, 7, 7) + 1, 3, quantum=0.5)
    _check(d, 14, 7, 7, -1000.25, [1, 777, 1 << 17], (1, 0))


@pytest.mark.parametrize("E0", [-100.25, 6.0])
@pytest.mark.parametrize("n,na,nb,ndets", [(12, 6, 6, 500), (12, 6, 2, 900), (12, 2, 6, 900), (34, 3, 3, 80), (34, 3, 1, 200)])
def test_threshold_over_batches(n, na, nb, ndets, E0):
    d = _case(n, na, nb, ndets, 60 + n + nb)
    pairs = _per(n, na, nb) * ndets
    for batches in (3, 9):
        _check(d, n, na, nb, E0, [1, 63, 64, 500, 5000], (1, 0), pair_buffer_bytes=(32 if n <= 32 else 48) * pairs // batches)
