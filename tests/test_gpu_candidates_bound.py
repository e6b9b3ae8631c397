"""candidates() in one pass into buffers for every pair against the pass that
counts first: the same tensors, bit for bit, and sized for what they hold."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,ndets,kw", [
    (10, 4, 4, 50, {}), (10, 4, 4, 50, {"ncore": 20}), (10, 4, 4, 50, {"ncore": 200}),
    (10, 4, 4, 50, {"eps": 1e-2}), (10, 4, 4, 50, {"pair_buffer_bytes": 1 << 16}), (36, 2, 3, 12, {}),
    (8, 8, 3, 6, {}), (6, 6, 6, 1, {}), (6, 6, 0, 1, {}), (5, 1, 0, 3, {}), (4, 2, 2, 36, {})])
def test_one_pass_equals_two(monkeypatch, n, na, nb, ndets, kw):
    import asci_synth as syn
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    rng = np.random.default_rng(5 * n + ndets)
    h, eri = syn.integrals(n, rng)
    dets = np.array(syn.uniform_dets(n, na, nb, ndets, rng), dtype=np.uint64)
    d = gu.to_dev({"h": h, "eri": eri, "dets": dets, "coeffs": syn.coefficients(ndets, ndets, rng)})
    got = []
    for _ in range(2):
        got.append(asci.candidates(d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], -2.0, **kw))
        monkeypatch.setattr(asci, "_pair_bound", lambda *a: 0)
    for one, two in zip(*got):
        assert one.shape == two.shape and (gu.host(one).view(np.uint64) == gu.host(two).view(np.uint64)).all()
        # (no candidates: the counting pass allocates one row)
        row = (2 if one.dim() == 2 else 1) * one.element_size()
        assert one.untyped_storage().nbytes() <= max(one.numel() * one.element_size(), row)


@pytest.mark.parametrize("short,kw,calls", [
    (None, {}, [1]),                                    # one pass
    ("library", {}, [1, 0, 1]),                         # the workspace did not fit beside the buffers
    ("torch", {}, [0, 1]),                              # the buffers did not fit
    ("copy", {}, [1, 0, 1]),                            # the copies did not fit beside them
    (None, {"pair_buffer_bytes": 1 << 16}, [0, 1])])    # the caller's pair buffer is smaller than the buffers
def test_counts_first_where_memory_is_short(monkeypatch, short, kw, calls):
    import torch

    import asci_synth as syn
    import gpu_util as gu
    import paper_2303_05688_amd as asci

    n, na, nb, ndets = 10, 4, 4, 50
    rng = np.random.default_rng(9)
    h, eri = syn.integrals(n, rng)
    dets = np.array(syn.uniform_dets(n, na, nb, ndets, rng), dtype=np.uint64)
    d = gu.to_dev({"h": h, "eri": eri, "dets": dets, "coeffs": syn.coefficients(ndets, ndets, rng)})
    args = (d["h"], d["eri"], n, na, nb, d["dets"], d["coeffs"], -2.0)
    want = [gu.host(t) for t in asci.candidates(*args)]
    bound = asci._pair_bound(n, na, nb, ndets, 0)
    real, empty, clone, seen = asci._lib.asci_candidates_device, torch.empty, torch.Tensor.clone, []

    def library(*a):
        seen.append(int(a[11] > 0))
        return asci.ASCI_ENOMEM if short == "library" and len(seen) == 1 else real(*a)

    def no_room(shape, **k):
        if shape[0] == bound:
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(shape, **k)

    def no_copy(t):
        raise torch.cuda.OutOfMemoryError("no room")

    monkeypatch.setattr(asci._lib, "asci_candidates_device", library)
    if short == "torch":
        monkeypatch.setattr(torch, "empty", no_room)
    if short == "copy":
        monkeypatch.setattr(torch.Tensor, "clone", no_copy)
    got = asci.candidates(*args, **kw)
    monkeypatch.setattr(torch.Tensor, "clone", clone)
    assert seen == calls
    for one, two in zip(got, want):
        assert (gu.host(one).view(np.uint64) == two.view(np.uint64)).all()
