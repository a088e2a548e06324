"""The one-launch MLP chain at the edges of its tiles (64 tokens, 16-token rows of them), for every width it is built for
and output widths off its 64-output steps."""
import dataclasses

import numpy as np
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dphi,d_emb,cache", [(64, 64, 512, True), (128, 128, 512, False), (128, 256, 512, True), (64, 128, 256, False),
                                                (128, 64, 256, True), (64, 64, 128, False), (128, 80, 512, False), (64, 16, 128, False)])
def test_chain_tile_edges(d, dphi, d_emb, cache):
    """Batch of mid-regions that end before, on and behind row and tile edges; budgets that put the retrieved rows there too
    (without a cache decode sends them through the same kernel).  Stored features, S, u, index sets and outputs
    against the float64 oracle, with the bounds of the stored features derived in parity_utils (2^-12 relative)."""
    import parity_utils as PU
    from oracle import tkphi_oracle as orc
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_q_heads=4, n_kv_heads=2, d_head=d, d_phi=dphi, seed=611)
    mids = [1, 15, 16, 17, 63, 64, 65, 200, 1500]
    ks = [1, 2, 15, 16, 17, 63, 64, 65, 129]
    layers = []
    for i, m in enumerate(mids):
        P = I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i)
        P["mlp"] = I.make_mlp_phi(w, layer=i, d_emb=d_emb)
        layers.append(P)
    b = H.Batch(H.config_of(w, cache_features=cache, d_emb=d_emb), layers, ks, debug=True)
    b.build()
    b.decode()
    assert b.status() & ~2 == 0          # (the residual clamp may fire where every mid token but one is retrieved)
    for i, (P, k) in enumerate(zip(layers, ks)):
        PU.check_layer(w, P, k, b, i)
        if cache:
            _, M = orc.partition(int(P["L"]), w.n_sink, w.n_tail)
            _, fk = PU.mlp_feature_fns(P)
            for h in range(w.n_kv_heads):
                F = fk[h](I.to_f64(P["K"])[h, M])
                rel = np.abs(b.result(i, "phi_cache")[h].astype(np.float64) - F) / F
                assert rel.max() <= PU.MLP_FEATURE_EPS, f"mid {mids[i]} head {h}: feature rel err {rel.max():.3e}"


@pytest.mark.parametrize("d,dphi,d_emb,mode", [(128, 128, 128, ""), (64, 128, 128, ""), (64, 64, 64, ""), (128, 128, 128, "unfused")])
def test_tied_weights(d, dphi, d_emb, mode):
    """Maps whose matrices are one buffer (Ws = W1 = W2 = Wo where the widths agree, else W1 = W2 = Wo): the packed copies of a
    matrix differ by the layer it serves, so the layer has to decide, not the address.  Against the float64 oracle, bounds
    as above."""
    import torch
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_q_heads=4, n_kv_heads=2, d_head=d, d_phi=dphi, seed=613)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 200)
    P["mlp"] = I.make_mlp_phi(w, layer=0, d_emb=d_emb)
    tied = [n for n, rows, cols in (("Ws", d_emb, d), ("W2", d_emb, d_emb), ("Wo", dphi, d_emb)) if (rows, cols) == (d_emb, d_emb)]
    assert "W2" in tied and len(tied) >= 2
    for side in ("q", "k"):
        for n in tied:
            P["mlp"][side][n] = P["mlp"][side]["W1"]
    b = H.Batch(H.config_of(w, cache_features=True, d_emb=d_emb, tuning={"mlp_mode": B.MLP_MODES[mode]}), [P], [40], debug=True)
    for side in ("q", "k"):                            # one buffer on the device as well
        t = b.dev[0][f"mlp_{side}_w"]
        for n in tied:
            t[n] = t["W1"]
        b.dev[0]["mlp_" + side].copy_(B.upload_mlp(t))
    torch.cuda.synchronize()
    b.build()
    b.decode()
    assert b.status() & ~2 == 0
    PU.check_layer(w, P, 40, b, 0)


@pytest.mark.parametrize("d,d_emb", [(128, 512), (64, 256), (64, 128)])
def test_large_output_bias_is_rounded_once(d, d_emb):
    """Output biases near -60: a sum that has the bias in it from the start rounds every one of its 2 d_emb / 32 steps at the ulp of
    60 (2^-18), one that takes it at the end rounds once.  The logarithm of a stored feature then carries what it carries
    with small biases (measured on the same weights), that one rounding (2^-19 / sqrt 3 rms) and the rounding of the
    bias itself and of exp's argument reduction in the float64 comparison (nothing and 2^-24 relative): 1.2 times the root of
    the sum of squares is allowed."""
    from oracle import tkphi_oracle as orc
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_q_heads=4, n_kv_heads=2, d_head=d, d_phi=d, seed=617)
    rms = []
    for shift in (0.0, -60.0):
        P = I.make_layer(w, L=w.n_sink + w.n_tail + 2000)
        P["mlp"] = I.make_mlp_phi(w, layer=0, d_emb=d_emb)
        P["mlp"]["k"]["bo"] = (P["mlp"]["k"]["bo"] + np.float32(shift)).astype(np.float32)
        b = H.Batch(H.config_of(w, cache_features=True, d_emb=d_emb), [P], [20])
        b.build()
        _, fk = PU.mlp_feature_fns(P)
        _, M = orc.partition(int(P["L"]), w.n_sink, w.n_tail)
        e = [np.log(b.result(0, "phi_cache")[h].astype(np.float64)) - np.log(fk[h](I.to_f64(P["K"])[h, M])) for h in range(w.n_kv_heads)]
        rms.append(float(np.sqrt(np.mean(np.square(e)))))
    print("log-feature error, rms:", d, d_emb, rms, flush=True)
    assert rms[1] <= 1.2 * np.hypot(rms[0], 2.0 ** -19 / np.sqrt(3.0)), rms


@pytest.mark.parametrize("d_emb,cache", [(128, True), (512, False), (1024, True)])
def test_hidden_units_far_outside(d_emb, cache):
    """Hidden biases of minus infinity and of -1e30 switch their units off (GeLU is zero there, not NaN): features, summaries and
    outputs are those of the maps whose second layer has zeros in these columns, on the chain, the layer-wise launches
    (d_emb 1024) and the query side."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_q_heads=4, n_kv_heads=2, d_head=64, d_phi=64, seed=619)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 300)
    P["mlp"] = I.make_mlp_phi(w, layer=0, d_emb=d_emb)
    O = dict(P, mlp={side: {n: t.copy() for n, t in P["mlp"][side].items()} for side in ("q", "k")})
    for side in ("q", "k"):
        P["mlp"][side]["b1"][:, [0, 17]], P["mlp"][side]["b1"][:, d_emb - 1] = -np.inf, -1e30
        O["mlp"][side]["W2"][:, :, [0, 17, d_emb - 1]] = 0
    b = H.Batch(H.config_of(w, cache_features=cache, d_emb=d_emb), [P], [40], debug=True)
    b.build()
    b.decode()
    assert b.status() & ~2 == 0
    PU.check_layer(w, O, 40, b, 0)


def test_recomputing_decode_replays_from_a_hip_graph():
    """A decode step without a feature cache (weight packing and the chain over the retrieved rows on the caller's stream, phi_q on
    the library's, 150 KB of LDS asked for at each launch) captured after one call outside, replayed with eager steps between:
    bit for bit the eager result."""
    import torch
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS["l3b_128k"]
    P = I.make_layer(w, L=3000)
    P["mlp"] = I.make_mlp_phi(w, d_emb=512)
    b = H.Batch(H.config_of(w, cache_features=False, d_emb=512), [P], [100], debug=True)
    b.build()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        b.decode()
        side.synchronize()
        eager = b.result(0, "out").copy()
        with torch.cuda.graph(graph, stream=side):
            b.decode()
    torch.cuda.synchronize()
    for _ in range(3):
        b.dev[0]["out"].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(b.result(0, "out"), eager)
        b.decode()
        torch.cuda.synchronize()
        assert np.array_equal(b.result(0, "out"), eager)


@pytest.mark.parametrize("d,d_emb,cache", [(128, 512, False), (128, 256, True), (64, 1024, True), (64, 128, False)])
@pytest.mark.parametrize("n_mid,k,select_test,chunk", [(700, 9, 0, 0), (9000, 600, 0, 0),       # short: scores in rows
                                                       (13003, 130, 0, 0), (13003, 900, 0, 0),  # bound handed over, one sweep of lists
                                                       (6000, 300, 1, 0), (6000, 300, 2, 0),    # rescan; every token a candidate
                                                       (2500, 0, 0, 256)])                      # nothing to retrieve
def test_one_problem_selects_lists(d, d_emb, cache, n_mid, k, select_test, chunk):
    """A decode step of one problem with MLP maps: filtered score pass, a workgroup per head that ends with the retrieved list, phi_q in
    the score and select launches (or the latter only, for short contexts), packed weights in the select launch, generated tokens behind
    the prefix.  Index sets, scores, outputs against the oracle; then the captured step, replayed with eager ones between, bit for
    bit."""
    import parity_utils as PU
    import torch
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_q_heads=6, n_kv_heads=2, d_head=d, d_phi=d, seed=733)
    n_gen = 70
    L = w.n_sink + w.n_tail + n_mid
    P = I.make_layer(w, L=L + n_gen)
    P["L"], P["n_gen"] = L, n_gen
    P["mlp"] = I.make_mlp_phi(w, layer=0, d_emb=d_emb)
    b = H.Batch(H.config_of(w, cache_features=cache, d_emb=d_emb, max_gen=80, tuning={"select_test": select_test, "scan_chunk": chunk}),
                [P], [k], debug=True)
    b.build()
    stages = dict(zip(B.STAGES, b.decode_stage_times()))
    assert stages["select"] > 0 and stages["select_plan"] == 0, stages
    assert b.status() & ~2 == 0
    PU.check_layer(w, P, k, b, 0)
    eager = b.result(0, "out").copy()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.decode()
    for _ in range(3):
        b.dev[0]["out"].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(b.result(0, "out"), eager)
        b.decode()
        torch.cuda.synchronize()
        assert np.array_equal(b.result(0, "out"), eager)
