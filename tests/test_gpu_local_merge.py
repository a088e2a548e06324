"""A head's only select workgroup merges it out of LDS; where retrieved indices are exported, or anchors fill more than six tiles of 64, the
merge goes by way of the workspace.  Both add the same partials in the same order: outputs agree bit for bit."""
import dataclasses

import numpy as np
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("dtype,d,mids,ks,tail,gen", [
    ("bf16", 64, [700], [50], 60, 0), ("bf16", 128, [700], [58], 60, 3), ("f32", 64, [700], [58], 60, 3),     # one tile and the edge of a second
    ("bf16", 64, [2000], [128], 317, 63), ("bf16", 64, [2000], [129], 317, 64),       # six tiles and one more; the edges of the split
    ("bf16", 128, [1600, 13, 90], [128, 1, 0], 60, 0),                                  # no retrieved tokens in one problem
    ("bf16", 64, [40000] * 9, [400] * 9, 60, 0), ("bf16", 128, [15000] * 12, [180] * 12, 60, 2)])      # lists, one workgroup per head
def test_local_merge(dtype, d, mids, ks, tail, gen, mode):
    import parity_utils as PU
    import torch
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype=dtype, n_q_heads=32, n_kv_heads=8, d_head=d, d_phi=d, n_sink=4, n_tail=tail, seed=97)
    layers = []
    for i, m in enumerate(mids):
        P = I.make_layer(w, L=4 + tail + m + gen, seq=i) if i < 3 else layers[i % 3]
        P["L"], P["n_gen"] = 4 + tail + m, gen
        layers.append(P)
    plain = H.Batch(H.config_of(w, max_gen=gen), layers, ks, max_K=max(ks))
    export = H.Batch(H.config_of(w, max_gen=gen), layers, ks, debug=True, max_K=max(ks))
    for b in (plain, export):
        b.build()
        b.decode(mode)
        b.decode(mode)                              # (the handed-over words are cleared as well)
        torch.cuda.synchronize()
        assert b.status() & ~2 == 0
    for i in range(len(mids)):
        y = plain.result(i, "out")
        assert np.isfinite(y).all() and np.array_equal(y, export.result(i, "out")), i
    if mode == 0 and max(mids) <= 2000:
        for i, (P, k) in enumerate(zip(layers, ks)):
            PU.check_layer(w, P, k, export, i, heads=[0, 31], sum_tol=2e-5)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("d,mid,ks,tail,gen", [
    (64, 3000, [1, 60, 128, 250, 0, 129], 60, 2), (64, 3000, [37], 317, 64),                  # 17 problems of 32 heads: 512 threads; scores by rows, six tiles and seven
    (64, 30000, [256, 300, 1, 511], 60, 0), (64, 30000, [300], 300, 10),                      # the same from lists
    (128, 2000, [128, 5], 60, 2), (128, 15000, [180, 0], 60, 2)])                             # 1024 threads
def test_local_merge_writes_aux(d, mid, ks, tail, gen, mode):
    """The same for a call that wants `aux` but no indices, which is merged out of LDS too, and for heads of the 512-thread kernel: outputs and
    aux agree bit for bit with the merge by way of the workspace, and with the oracle at the bars of parity_utils."""
    import parity_utils as PU
    import torch
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype="bf16", n_q_heads=32, n_kv_heads=8, d_head=d, d_phi=d, n_sink=4, n_tail=tail, seed=97)
    n = 17
    base = [I.make_layer(w, L=4 + tail + mid + gen, seq=i) for i in range(2)]
    for P in base:
        P.update(L=4 + tail + mid, n_gen=gen)
    layers, kk = [base[i % 2] for i in range(n)], [ks[i % len(ks)] for i in range(n)]
    plain = H.Batch(H.config_of(w, max_gen=gen), layers, kk)
    with_aux = H.Batch(H.config_of(w, max_gen=gen), layers, kk, debug=True)
    export = H.Batch(H.config_of(w, max_gen=gen), layers, kk, debug=True)
    for i in range(n):
        with_aux.host_table[i].topk_idx = None
        with_aux.dev[i]["topk_idx"].fill_(-5)
        with_aux.dev[i]["aux"].fill_(float("nan"))
    with_aux.set_topk(0, kk[0])                         # (uploads the table)
    for b in (plain, with_aux, export):
        b.build()
        b.decode(mode)
        torch.cuda.synchronize()
        assert b.status() & ~2 == 0
    for i in range(n):
        y = plain.result(i, "out")
        assert np.isfinite(y).all() and np.array_equal(y, export.result(i, "out")) and np.array_equal(y, with_aux.result(i, "out")), i
        assert np.array_equal(with_aux.result(i, "aux"), export.result(i, "aux")), i
        assert (with_aux.result(i, "topk_idx") == -5).all()
    if mode == 0 and mid <= 3000:
        for i in range(0, min(n, 2 * len(ks)), 2 if len(ks) == 1 else 1):
            PU.check_layer(w, layers[i], kk[i], export, i, heads=[0, 31], sum_tol=2e-5)


@pytest.mark.parametrize("d,ks", [(64, [256, 257, 511, 512, 513, 1024, 1025, 1536, 1600]), (64, [255, 256, 257, 511, 512, 513, 700, 1023, 1024] * 2),
                                  (128, [255, 256, 257, 511, 512, 513, 1024, 1536, 1600])])
def test_gather_rounds(d, ks):
    """One workgroup per head, winners around the rounds, against the oracle at the bars of parity_utils: 9 problems of 32 heads, rounds of 512
    (d = 64) or 256, and beyond the 1536 winners kept in LDS; 18 problems at d = 64 and at most 1024 winners, all of which are kept: the
    512-thread kernel and its rounds of 256."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype="bf16", n_q_heads=32, n_kv_heads=8, d_head=d, d_phi=d, seed=98)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 20001)
    b = H.Batch(H.config_of(w), [P] * len(ks), ks, debug=True)
    b.build()
    b.decode()
    assert b.status() & ~2 == 0
    for i, k in enumerate(ks):
        PU.check_layer(w, P, k, b, i, heads=[i], sum_tol=2e-5)
