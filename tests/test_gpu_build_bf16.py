"""The bf16 matrix-core summary build at the edges of its tiles (32 tokens, dealt to the wavefronts of a workgroup in turn) and chunks, both
head dimensions, with strides of its own and rows that lie apart."""
import dataclasses

import numpy as np
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu

MIDS = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 97, 127, 128, 129, 255, 257, 300, 383, 385, 1000]


@pytest.mark.parametrize("cache", [False, True])
@pytest.mark.parametrize("d,chunk", [(64, 0), (64, 64), (64, 192), (64, 512), (128, 0), (128, 64)])
def test_build_bf16_edges(d, chunk, cache):
    """S, u (and the cached features) against the float64 oracle.  A feature enters S as 16 bits (2^-17) and its exponent carries
    |logit| 2^-23 of the fp32 products: 2e-5 of either, the bar of the other builds."""
    import parity_utils as PU
    from oracle import tkphi_oracle as orc
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype="bf16", n_q_heads=4, n_kv_heads=2, d_head=d, d_phi=d, seed=95)
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i) for i, m in enumerate(MIDS)]
    for sel in ([slice(0, len(MIDS))] if cache else [slice(0, len(MIDS)), slice(7, 8), slice(20, 21)]):
        b = H.Batch(H.config_of(w, cache_features=cache, tuning={"build_chunk": chunk}), layers[sel], [1] * len(layers[sel]), debug=True)
        b.build()
        assert b.status() == 0
        for i, P in enumerate(layers[sel]):
            O = PU.oracle_inputs(P)
            S, u = orc.build_summaries(O["K"], O["V"], O["Wk"], O["bk"], w.phi_in_scale, w.phi_norm_coef, w.n_sink, w.n_tail)
            PU.check_summaries(b.result(i, "S"), b.result(i, "u"), S, u, 2e-5)
            if cache:
                _, M = orc.partition(int(P["L"]), w.n_sink, w.n_tail)
                for h in range(w.n_kv_heads):
                    F = orc.phi(O["K"][h, M], O["Wk"][h], O["bk"][h], w.phi_in_scale, w.phi_norm_coef)
                    rel = np.abs(b.result(i, "phi_cache")[h].astype(np.float64) - F) / F
                    assert rel.max() <= 2e-5, f"mid {MIDS[i]} head {h}: feature rel err {rel.max():.3e}"


@pytest.mark.parametrize("c", [0.0, 0.05])
def test_build_bf16_strided(c):
    """Rows of three times their length (K and V interleaved with a third tensor, heads behind each other) give what contiguous
    rows give, bit for bit, and a norm coefficient of 0 is no special case."""
    import torch
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype="bf16", n_q_heads=2, n_kv_heads=2, d_head=64, d_phi=64, seed=96)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 701)
    cfg = H.config_of(w)
    cfg.phi_norm_coef = c
    plain = H.Batch(cfg, [P], [1])
    plain.build()
    K, V = plain.dev[0]["K"], plain.dev[0]["V"]
    big = torch.full((K.shape[0], K.shape[1], 3, 64), float("nan"), dtype=K.dtype, device="cuda")
    big[:, :, 0], big[:, :, 2] = K, V
    apart = H.Batch(cfg, [dict(P, K=big[:, :, 0], V=big[:, :, 2])], [1])
    apart.build()
    assert plain.status() == 0 and apart.status() == 0
    for name in ("S", "u"):
        x = plain.result(0, name)
        assert np.isfinite(x).all() and np.array_equal(x, apart.result(0, name))


@pytest.mark.parametrize("dtype,d,hkv,n,L,longer", [("bf16", 64, 8, 1, 10126, 11539), ("bf16", 64, 8, 1, 8212, 15593), ("bf16", 128, 1, 2, 8000, 0),
                                                      ("f32", 64, 8, 1, 6000, 0)])
def test_build_in_a_smaller_workspace(dtype, d, hkv, n, L, longer):
    """Builds that take fewer chunks than they would like, as their workspace is that of longer sequences (or half their own): S and u against
    the float64 oracle at the bars of test_build_bf16_edges, and nothing behind the end of the workspace is written."""
    import parity_utils as PU
    import torch
    from oracle import tkphi_oracle as orc
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype=dtype, n_q_heads=hkv, n_kv_heads=hkv, d_head=d, d_phi=d, seed=99)
    layers = [I.make_layer(w, L=L, seq=i) for i in range(n)]
    b = H.Batch(H.config_of(w), layers, [L // 100] * n)
    have = B.tkphi_workspace_bytes(b.cfg, n, longer, longer // 100) if longer else b.ws_bytes // 2 // 256 * 256
    assert 0 < have < b.ws_bytes
    guard = 1 << 20
    ws = torch.full((have + guard,), 0x5a, dtype=torch.uint8, device="cuda")
    B.tkphi_build_summaries(b.cfg, b.table.data_ptr(), n, L, ws.data_ptr(), have, B.current_stream_ptr())
    torch.cuda.synchronize()
    assert bool((ws[have:] == 0x5a).all())
    for i, P in enumerate(layers):
        O = PU.oracle_inputs(P)
        S, u = orc.build_summaries(O["K"], O["V"], O["Wk"], O["bk"], w.phi_in_scale, w.phi_norm_coef, w.n_sink, w.n_tail)
        PU.check_summaries(b.result(i, "S"), b.result(i, "u"), S, u, 2e-5)


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64)])
def test_biases_need_no_alignment(dtype, d):
    """bk and bq as they may lie inside a larger fp32 buffer, 4, 8 and 12 bytes past a 16-byte boundary: S, u and the step's output keep their bits."""
    import torch
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype=dtype, n_q_heads=4, n_kv_heads=2, d_head=d, d_phi=d, seed=94)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 500)
    rng = np.random.default_rng(7)
    P["bk"] = rng.standard_normal(P["bk"].shape).astype(np.float32)
    P["bq"] = np.repeat(P["bk"], 2, axis=0)
    b = H.Batch(H.config_of(w), [P], [9])
    b.build()
    b.decode()
    want = {name: b.result(0, name) for name in ("S", "u", "out")}
    for off in (1, 2, 3):
        keep = {}
        for name in ("bk", "bq"):
            t = b.dev[0][name].flatten()
            keep[name] = torch.full((t.numel() + 8,), float("nan"), dtype=torch.float32, device="cuda")
            keep[name][off:off + t.numel()] = t
            setattr(b.host_table[0], name, keep[name].data_ptr() + 4 * off)
        for name in want:
            b.dev[0][name].zero_()
        b.set_topk(0, 9)                                # (uploads the table)
        b.build()
        b.decode()
        torch.cuda.synchronize()
        for name, x in want.items():
            assert np.isfinite(x).all() and np.array_equal(b.result(0, name), x), (off, name)


@pytest.mark.parametrize("cache", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_infinite_and_undefined_rows(d, cache):
    """What keys and values that are infinite or no numbers reach, and nothing else: a row is contracted into S and u of its own head, a value only
    into its channel, rows outside the mid-region into nothing.  (fp32 exponents: a key whose squared norm overflows has features 0 if its products stay finite.)"""
    import torch
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype="bf16", n_q_heads=3, n_kv_heads=3, d_head=d, d_phi=d, seed=93)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 1000)
    cfg = H.config_of(w, cache_features=cache)
    clean = H.Batch(cfg, [P], [1])
    clean.build()
    S, u = clean.result(0, "S"), clean.result(0, "u")
    assert np.isfinite(S).all() and np.isfinite(u).all()
    inf, nan = float("inf"), float("nan")
    last = w.n_sink + 999                               # the last row of the mid-region, which the padding of a tile repeats

    def build(edit):
        K, V = clean.dev[0]["K"].clone(), clean.dev[0]["V"].clone()
        edit(K, V)
        b = H.Batch(cfg, [dict(P, K=K, V=V)], [1])
        b.build()
        torch.cuda.synchronize()
        assert b.status() == 0
        return b.result(0, "S"), b.result(0, "u")

    for tok in (w.n_sink, w.n_sink + 517, last):
        for x in (inf, -inf, nan):
            def value(K, V):
                V[1, tok, 5] = x
            Sx, ux = build(value)
            assert np.array_equal(ux, u) and np.array_equal(Sx[[0, 2]], S[[0, 2]])
            rest = [c for c in range(d) if c != 5]
            assert np.array_equal(Sx[1][:, rest], S[1][:, rest]) and not np.isfinite(Sx[1][:, 5]).any()

            def key(K, V):
                K[1, tok, 5] = x
            Sx, ux = build(key)
            assert np.array_equal(ux[[0, 2]], u[[0, 2]]) and np.array_equal(Sx[[0, 2]], S[[0, 2]])
            if x != x:
                assert np.isnan(ux[1]).all() and np.isnan(Sx[1]).all()
    # rows outside the mid-region
    def outside(K, V):
        for t in (K, V):
            t[:, :w.n_sink] = nan
            t[:, last + 1:] = inf
    Sx, ux = build(outside)
    assert np.array_equal(Sx, S) and np.array_equal(ux, u)

    # a row of norm^2 beyond fp32, its products with W finite: features of exp(-inf) = 0, as if the row were not there
    def huge(K, V):
        K[1, w.n_sink + 517] = 2.0 ** 64
    def gone(K, V):
        K[1, w.n_sink + 517] = 64.0                     # (|k|^2 / (2 sqrt d) in the thousands: exp underflows)
    Sh, uh = build(huge)
    Sg, ug = build(gone)
    assert np.array_equal(Sh, Sg) and np.array_equal(uh, ug) and np.isfinite(Sh).all()
