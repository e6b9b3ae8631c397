"""Searches of one small class batch (read back once, at the end) against the
step-by-step path, which candidates() takes: the k largest of every candidate
in exact (|A| descending, key ascending) order, bit for bit, on both sides of
each rule (one split level up to 2^19 pairs, two above; a sort of every
candidate up to 2^20, a selection above; the step-by-step path from 2^22), with k at the edges of the sort's chunks,
and among scores of which most are tied.  The same errors on both paths."""
from math import comb

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pairs(n, na, nb):
    va, vb = n - na, n - nb
    return (na * va + nb * vb + comb(na, 2) * comb(va, 2) + comb(nb, 2) * comb(vb, 2) + na * va * nb * vb)


def _case(n, na, nb, ndets, seed, quantum=None):
    import asci_synth as syn

    rng = np.random.default_rng(seed)
    h, eri = syn.integrals(n, rng)
    dets = np.array(syn.uniform_dets(n, na, nb, ndets, rng), dtype=np.uint64)
    c = syn.coefficients(ndets, ndets, rng)
    if quantum is not None:  # sums of few multiples of a power of two: many exact ties, many exact zeros
        h, eri = np.round(h / quantum) * quantum, np.round(eri / quantum) * quantum
        c = np.sign(c + 1e-30) * 2.0 ** -np.ceil(np.log2(ndets) / 2)
    return {"h": h, "eri": eri, "dets": dets, "coeffs": c}


def _expected(d, n, na, nb, E0, **kw):
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    k, _, sc = (gu.host(x) for x in asci.candidates(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], E0, **kw))
    order = np.lexsort((k[:, 1], k[:, 0], ~gu.abs_bits(sc)))
    return k[order], sc[order]


def _compare(d, n, na, nb, E0, ks, want, **kw):
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    for k in ks:
        gk, gs = (gu.host(x) for x in asci.search(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], E0, k, **kw))
        m = min(k, len(want[1]))
        assert len(gs) == m, (k, len(gs), m)
        assert (gk == want[0][:m]).all() and (gs.view(np.uint64) == want[1][:m].view(np.uint64)).all(), k


@pytest.mark.parametrize("n,na,nb", [(12, 6, 6), (34, 3, 3)])
@pytest.mark.parametrize("log_pairs,over", [(12, 0), (19, 0), (19, 1), (20, 0), (20, 1), (22, 0), (22, 1)])
def test_small_search_edges(n, na, nb, log_pairs, over):
    import gpu_util as gu

    nd = max((1 << log_pairs) // _pairs(n, na, nb) + over, 1)
    d = gu.to_dev(_case(n, na, nb, nd, 900 + n + log_pairs))
    want = _expected(d, n, na, nb, -3.5)
    ks = [1, 1023, 1024, 1025, 4097, len(want[1]) - 1, len(want[1]), len(want[1]) + 1]
    _compare(d, n, na, nb, -3.5, [k for k in ks if k > 0], want)
    for kw in ({"ncore": (nd + 1) // 2}, {"eps": 1e-3}, {"constraint_level": 1}, {"constraint_level": 5}):
        _compare(d, n, na, nb, -3.5, [500], _expected(d, n, na, nb, -3.5, **kw), **kw)


@pytest.mark.parametrize("n,na,nb,ndets", [(12, 6, 6, 40), (12, 6, 6, 300), (34, 3, 3, 60)])
def test_small_search_tied_scores(n, na, nb, ndets):
    import gpu_util as gu

    d = gu.to_dev(_case(n, na, nb, ndets, 31 + ndets, quantum=0.5))
    want = _expected(d, n, na, nb, -1000.25)
    assert len(np.unique(gu.abs_bits(want[1]))) < len(want[1]) // 2
    _compare(d, n, na, nb, -1000.25, [1, 2, 1024, 1025, 2049, 8193, len(want[1]) - 1, len(want[1])], want)


@pytest.mark.parametrize("n,na,nb", [(12, 6, 6), (34, 3, 3)])
@pytest.mark.parametrize("fault", ["electrons", "duplicate", "eri"])
def test_small_search_errors(n, na, nb, fault):
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    good = _case(n, na, nb, 24, 7)
    bad = {k: v.copy() for k, v in good.items()}
    if fault == "electrons":
        bad["dets"][11, 0] = (1 << (na + 1)) - 1
    elif fault == "duplicate":
        bad["dets"][23] = bad["dets"][2]
    else:
        bad["eri"].reshape(n, n, n, n)[0, 1, 2, 3] += 1e-3
    said = []
    for kw in ({}, {"pair_buffer_bytes": 32 * 12 * _pairs(n, na, nb)}):  # the second: several batches
        d = gu.to_dev(bad)
        with pytest.raises(asci.AsciError) as e:
            asci.search(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], -3.5, 100, **kw)
        said.append((e.value.code if hasattr(e.value, "code") else None, str(e.value)))
    assert said[0] == said[1]
    d = gu.to_dev(good)
    _compare(d, n, na, nb, -3.5, [100], _expected(d, n, na, nb, -3.5))


@pytest.mark.parametrize("n,na,nb", [(12, 6, 6), (9, 3, 2), (34, 3, 3)])
@pytest.mark.parametrize("alpha,beta", [(0, 0), (1, 1), ("all", "all"), ("more", 0), (0, "more"), ("high", 1), (1, "high")])
def test_small_search_invalid_strings(n, na, nb, alpha, beta):
    """Strings with too few, too many or outside orbitals, in the core set: the
    search reads its flags at the end, so it runs on what takes their place."""
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    mask = {"all": (1 << n) - 1, "more": (1 << (max(na, nb) + 2)) - 1, "high": (1 << 63) | (1 << n)}
    good = _case(n, na, nb, 24, 11)
    bad = {k: v.copy() for k, v in good.items()}
    for i in (0, 5, 23):
        bad["dets"][i] = (np.uint64(mask.get(alpha, alpha)), np.uint64(mask.get(beta, beta)))
    d = gu.to_dev(bad)
    for kw in ({}, {"ncore": 10}):
        with pytest.raises(asci.AsciError) as e:
            asci.search(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], -3.5, 100, **kw)
        assert e.value.code == asci.ASCI_EINVAL
    d = gu.to_dev(good)
    _compare(d, n, na, nb, -3.5, [100], _expected(d, n, na, nb, -3.5))


@pytest.mark.parametrize("n,na,nb,ndets", [(14, 13, 6, 948), (10, 8, 5, 3780), (16, 1, 8, 2146), (16, 2, 8, 380),
                                           (34, 33, 2, 1200)])
def test_small_search_dense_space(n, na, nb, ndets):
    """Targets with hundreds of contributions each, so that a small split's
    ranges of several keys exceed a wavefront's share: they are divided where
    they arise, for every finish capacity, and no further level is taken."""
    import asci_synth as syn
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    assert ndets * _pairs(n, na, nb) <= 1 << 22
    rng = np.random.default_rng(n + ndets)
    h, eri = syn.integrals(n, rng)
    dets = np.array(syn.level_dets(n, na, nb, ndets, rng), dtype=np.uint64)
    d = gu.to_dev({"h": h, "eri": eri, "dets": dets, "coeffs": syn.coefficients(ndets, ndets, rng)})
    want = None
    for cap in (4096, 2048, 1024):
        ctx = asci.Context(0)
        ctx.set_param("finish_cap", cap)
        every = _expected(d, n, na, nb, -3.5, ctx=ctx)
        want = want or every
        assert (every[0] == want[0]).all() and (every[1].view(np.uint64) == want[1].view(np.uint64)).all()
        _compare(d, n, na, nb, -3.5, [1, 1025, 4000], want, ctx=ctx)
        assert ctx.get_param("last_levels") <= 2
        r = asci.SearchRequest(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], -3.5, 4000)
        count, status, flags = asci.async_status(asci.search_async(r, ctx=ctx))
        assert (status, flags) == (0, 0)
        gk, gs = (gu.host(x) for x in r.result(count))
        m = min(4000, len(want[1]))
        assert count == m and (gk == want[0][:m]).all() and (gs.view(np.uint64) == want[1][:m].view(np.uint64)).all()
        ctx.close()


@pytest.mark.parametrize("n,na,nb,ndets", [(12, 4, 4, 201), (12, 6, 6, 2300), (16, 8, 2, 1500), (34, 3, 3, 360)])
def test_small_search_holds_no_more_than_the_steps(n, na, nb, ndets):
    """Device memory that a context keeps after a small search: no more than
    after the step-by-step search of the same inputs (profiling takes it)."""
    import gpu_util as gu
    import paper_2303_05688_amd as asci
    import torch

    assert ndets * _pairs(n, na, nb) <= 1 << 22
    d = gu.to_dev(_case(n, na, nb, ndets, 5))
    held = []
    for steps in (True, False, True, False):  # the first two load the kernels
        ctx = asci.Context(0)
        ctx.set_profiling(steps)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info(0)[0]
        asci.search(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], -3.5, 10 * ndets, ctx=ctx)
        torch.cuda.synchronize()
        held.append(before - torch.cuda.mem_get_info(0)[0])
        ctx.close()
    print("held", held)
    assert 0 < held[3] <= held[2]
