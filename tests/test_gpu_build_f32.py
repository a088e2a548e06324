"""The fp32-arithmetic summary build at the edges of its tiles (64 tokens, 16-token rows of them), feature tiles per
wavefront (d_phi up to 64, 128, 256, off multiples of 64) and chunks, both storage types and head dimensions."""
import dataclasses

import numpy as np
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cache", [False, True])
@pytest.mark.parametrize("dtype,d,dphi,chunk", [("f32", 64, 64, 0), ("f32", 64, 16, 128), ("f32", 128, 80, 64), ("f32", 128, 256, 192),
                                                ("bf16", 64, 128, 64), ("bf16", 128, 48, 0), ("bf16", 64, 192, 128)])
def test_build_f32_edges(dtype, d, dphi, chunk, cache):
    """S, u (and the cached features) of a batch whose mid-regions end on, before and behind every kind of edge, against the
    float64 oracle: relative Frobenius error 2e-5, the bar of the fp32 arithmetic (fp32 sums of at most 4096 tokens per
    chunk; a feature's exponent carries |logit| 2^-23, below 1e-5 for the logits of these inputs)."""
    import parity_utils as PU
    from oracle import tkphi_oracle as orc
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype=dtype, n_q_heads=4, n_kv_heads=2, d_head=d, d_phi=dphi, seed=91)
    mids = [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 300, 1000]
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i) for i, m in enumerate(mids)]
    b = H.Batch(H.config_of(w, cache_features=cache, tuning={"build_chunk": chunk}), layers, [1] * len(layers), debug=True)
    b.build()
    assert b.status() == 0
    for i, P in enumerate(layers):
        O = PU.oracle_inputs(P)
        S, u = orc.build_summaries(O["K"], O["V"], O["Wk"], O["bk"], w.phi_in_scale, w.phi_norm_coef, w.n_sink, w.n_tail)
        PU.check_summaries(b.result(i, "S"), b.result(i, "u"), S, u, 2e-5)
        if cache:
            _, M = orc.partition(int(P["L"]), w.n_sink, w.n_tail)
            for h in range(w.n_kv_heads):
                F = orc.phi(O["K"][h, M], O["Wk"][h], O["bk"][h], w.phi_in_scale, w.phi_norm_coef)
                rel = np.abs(b.result(i, "phi_cache")[h].astype(np.float64) - F) / F
                assert rel.max() <= 2e-5, f"mid {mids[i]} head {h}: feature rel err {rel.max():.3e}"


@pytest.mark.parametrize("dtype,d,dphi", [("f32", 64, 64), ("f32", 128, 16), ("f32", 128, 256), ("bf16", 64, 80), ("bf16", 128, 48)])
def test_gather_f32_edges(dtype, d, dphi):
    """Decode on the fp32-arithmetic kernels: retrieved counts around the 16-token rows and 64-token tiles of the gather, feature
    widths of an odd and an even number of 16-feature tiles, mid-regions that make the score pass run with 256 and (few
    workgroups) 1024 threads.  The bars of parity_utils: scores 1e-5, outputs 2e-3, residual terms 1e-4."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype=dtype, n_q_heads=6, n_kv_heads=2, d_head=d, d_phi=dphi, seed=92)
    ks = [1, 15, 16, 17, 63, 64, 65, 129]
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + 300 + 211 * i, seq=i) for i in range(len(ks))]
    for sel in (slice(0, 8), slice(6, 7)):
        b = H.Batch(H.config_of(w), layers[sel], ks[sel], debug=True)
        b.build()
        b.decode()
        assert b.status() == 0
        for i, (P, k) in enumerate(zip(layers[sel], ks[sel])):
            PU.check_layer(w, P, k, b, i, sum_tol=2e-5)


@pytest.mark.parametrize("hq,hkv", [(1, 1), (6, 2), (8, 1)])
@pytest.mark.parametrize("mids,ks", [([12], [1]), ([127], [10]), ([128], [10]), ([129], [9]), ([12288], [1024]), ([12289], [300]),
                                     ([4000, 13, 700], [257, 1, 50]), ([3100, 200, 12288], [258, 16, 100])])
def test_short_f32_contexts(hq, hkv, mids, ks):
    """Short fp32 contexts at d = d_phi = 64: two launches up to a budget of 1/12 and 12288 mid tokens (beyond: six), over the edges of
    the score workgroups' 128 rows, several workgroups per head, one and several gather rounds of 256, ties, generated tokens.
    Scores, index sets and outputs against the oracle at the bars of parity_utils; the captured step replays bit for bit."""
    import parity_utils as PU
    import torch
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], n_q_heads=hq, n_kv_heads=hkv, seed=93)
    layers = []
    for i, m in enumerate(mids):
        P = I.make_layer(w, L=w.n_sink + w.n_tail + m + 5, seq=i)
        P["L"], P["n_gen"] = w.n_sink + w.n_tail + m, 5
        if m >= 127:
            P["K"][:, w.n_sink + m // 2:w.n_sink + m // 2 + 6] = P["K"][:, w.n_sink + 3:w.n_sink + 4]        # equal scores
        layers.append(P)
    b = H.Batch(H.config_of(w, max_gen=8), layers, ks, debug=True)
    b.build()
    stages = dict(zip(B.STAGES, b.decode_stage_times()))
    assert (stages["select"] > 0) == (max(mids) <= 12288 and max(ks) * 12 <= max(mids)), stages
    assert b.status() & ~2 == 0
    for i, (P, k) in enumerate(zip(layers, ks)):
        PU.check_layer(w, P, k, b, i, heads=sorted({0, hq // 2, hq - 1}), sum_tol=2e-5)
    eager = [b.result(i, "out").copy() for i in range(len(mids))]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.decode()
    for _ in range(3):
        for i in range(len(mids)):
            b.dev[i]["out"].zero_()
        graph.replay()
        torch.cuda.synchronize()
        for i in range(len(mids)):
            assert np.array_equal(b.result(i, "out"), eager[i])
        b.decode()
        torch.cuda.synchronize()
