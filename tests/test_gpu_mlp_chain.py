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
