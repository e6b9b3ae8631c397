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
