"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Sizes here span several tiles / slices and ragged tails while the oracle
still finishes in seconds; the full-size workloads are in test_gpu_fullsize.py."""
import dataclasses

import numpy as np
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


def _batch(w, layers, topk, cache_features=False, tuning=None, **kw):
    from paper_2604_05438_amd import harness as H
    return H.Batch(H.config_of(w, cache_features=cache_features, tuning=tuning), layers, topk, debug=True, **kw)


def _run_single(w, L, k, mode="sub", heads=None, **kw):
    from paper_2604_05438_amd import binding as B
    import parity_utils as PU
    P = I.make_layer(w, L=L)
    b = _batch(w, [P], [k], **kw)
    b.build()
    b.decode({"sub": B.TKPHI_MODE_SUB, "nosub": B.TKPHI_MODE_NOSUB, "topk": B.TKPHI_MODE_TOPK_ONLY}[mode])
    st = b.status()
    assert st == 0, f"device status {st}"
    return PU.check_layer(w, P, k, b, 0, heads=heads, mode=mode), b, P


def test_tiny_f32_config():
    # Tiny single head, fp32: L 4096, 4 sink + 64 tail, K = 40, d = d_phi = 64
    w = I.WORKLOADS["tiny_f32"]
    k = I.mid_budget(w.L, w.budget_bp, w.n_sink, w.n_tail)
    assert k == 40
    rep, _, _ = _run_single(w, w.L, k)
    print("tiny_f32", rep)


@pytest.mark.parametrize("L,k", [(2500, 24), (777, 7), (5000, 49), (4229, 300)])
def test_l1b_shape_small(L, k):
    # 32 query / 8 KV heads (GQA 4:1), head_dim 64, bf16; ragged lengths
    w = I.WORKLOADS["l1b_32k"]
    rep, _, _ = _run_single(w, L, k)
    print("l1b", L, k, rep)


@pytest.mark.parametrize("L,k", [(3001, 29), (9000, 360)])
def test_l3b_shape_small(L, k):
    # 24 query / 8 KV heads (GQA 3:1), head_dim 128, bf16
    w = I.WORKLOADS["l3b_128k"]
    rep, _, _ = _run_single(w, L, k)
    print("l3b", L, k, rep)


@pytest.mark.parametrize("shape", ["l3b_128k", "l1b_32k"])
@pytest.mark.parametrize("chunk", [64, 128, 2048])
def test_build_tile_and_chunk_boundaries(shape, chunk):
    """Summary build alone (eq. (natural_cache)) at mid-region sizes around the boundaries of its tiling: one token,
    one short of / exactly / one past a 32-token tile, the same around the chunk size (a workgroup then sees 1 to 5
    tiles: fewer than, as many as and more than the stages of its LDS ring) and several chunks with a ragged last
    one; chunk = 64 and 128 force those small chunks, 2048 is the size long sequences use.  A batch of all lengths
    in one call; S and u of every KV head against the oracle under the bf16-feature bound."""
    import parity_utils as PU
    from oracle import tkphi_oracle as orc
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    edge = w.n_sink + w.n_tail
    mids = sorted({1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 4 * chunk - 1, 4 * chunk, 4 * chunk + 33})
    mids = [m for m in mids if m <= 8300]
    layers = [I.make_layer(w, L=edge + m, seq=i) for i, m in enumerate(mids)]
    b = H.Batch(H.config_of(w, tuning={"build_chunk": chunk}), layers, [1] * len(layers), debug=True)
    b.build()
    assert b.status() == 0
    for i, (P, m) in enumerate(zip(layers, mids)):
        O = PU.oracle_inputs(P)
        S_or, u_or = orc.build_summaries(O["K"], O["V"], O["Wk"], O["bk"], w.phi_in_scale, w.phi_norm_coef, w.n_sink, w.n_tail)
        PU.check_summaries(b.result(i, "S"), b.result(i, "u"), S_or, u_or, 2e-3, w=w, O=O)
    print("build boundaries", shape, chunk, mids, flush=True)


@pytest.mark.parametrize("shape,L,k,d_emb", [("l3b_128k", 9000, 90, 0), ("l3b_128k", 5000, 600, 0), ("l1b_32k", 5000, 49, 0),
                                             ("f32_gqa", 2000, 20, 0), ("l1b_32k", 3000, 29, 128)])
def test_token_major_cache_layout(shape, L, k, d_emb):
    """K and V stored token-major ([token][KV head][channel], the layout of a cache that appends one row of all
    heads per step): the library sees it through stride_head = d and stride_tok = Hkv d.  Every kernel that walks
    key or value rows (build tiles, score scan, sample, gather, anchors, the MLP stem) takes the strides from the
    problem record; results must equal the head-major run of the same data, which the oracle checks."""
    import torch
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    if shape == "f32_gqa":                                       # generic kernels: fp32 storage, GQA 2:1, d_phi != d_head
        w = dataclasses.replace(I.WORKLOADS["tiny_f32"], n_q_heads=4, n_kv_heads=2, d_head=128, d_phi=48, name="f32_gqa", seed=79)
    else:
        w = I.WORKLOADS[shape]
    P = I.make_layer(w, L=L)
    if d_emb:
        P["mlp"] = I.make_mlp_phi(w, layer=0, d_emb=d_emb)
    dev = dict(P)
    for name in ("K", "V"):
        hm = H.to_device(P[name])                               # [Hkv][L][d]
        dev[name] = hm.permute(1, 0, 2).contiguous().permute(1, 0, 2)
        assert dev[name].stride() == (w.d_head, w.n_kv_heads * w.d_head, 1) and torch.equal(dev[name], hm)
    b = H.Batch(H.config_of(w, d_emb=d_emb), [dev], [k], debug=True)
    b.build(); b.decode()
    assert b.status() == 0
    print("token-major", shape, L, k, PU.check_layer(w, P, k, b, 0), flush=True)


@pytest.mark.parametrize("shape,L,k,chunk", [("l3b_128k", 20011, 200, 1024), ("l1b_32k", 9000, 90, 2048),
                                             ("l3b_128k", 5000, 600, 512)])
def test_interleaved_chunks(shape, L, k, chunk):
    """The chunk-to-row mapping used for long single sequences (every workgroup takes every
    n_chunks-th unit of 256 / 512 rows), forced here at sizes the oracle checks in full; ragged
    last units, and a single problem as well as a ragged batch."""
    import parity_utils as PU
    tuning = {"interleave": 1, "scan_chunk": chunk}
    w = I.WORKLOADS[shape]
    rep, _, _ = _run_single(w, L, k, tuning=tuning)
    print("interleaved", shape, L, k, rep)
    Ls = [L, L // 2 + 3, 700]
    ks = [k, 11, 5]
    layers = [I.make_layer(w, L=l, seq=i) for i, l in enumerate(Ls)]
    b = _batch(w, layers, ks, tuning=tuning)
    b.build(); b.decode()
    assert b.status() == 0
    for i, (P, kk) in enumerate(zip(layers, ks)):
        PU.check_layer(w, P, kk, b, i, heads=[0, w.n_q_heads // 2, w.n_q_heads - 1])


@pytest.mark.parametrize("mode", ["nosub", "topk"])
def test_accounting_variants(mode):
    w = I.WORKLOADS["l1b_32k"]
    rep, _, _ = _run_single(w, 3000, 29, mode=mode)
    print(mode, rep)


def test_generic_kernels_forced_on_a_matrix_core_shape():
    """tkphi_tuning::force_generic: the fp32-arithmetic kernels on bf16 storage with d_phi == d_head."""
    w = I.WORKLOADS["l1b_32k"]
    rep, _, _ = _run_single(w, 2100, 21, heads=[0, 9, 31], tuning={"force_generic": 1})
    print("forced generic", rep)


def test_f32_gqa_and_dphi_not_equal_d():
    # generic path: fp32 storage, GQA 2:1, d_phi != d_head
    w = dataclasses.replace(I.WORKLOADS["tiny_f32"], n_q_heads=4, n_kv_heads=2, d_head=128, d_phi=48,
                            name="f32_gqa", seed=77)
    rep, _, _ = _run_single(w, 1500, 33)
    print("f32 gqa", rep)


def test_degenerate_budgets_and_lengths():
    """K = 0; K >= |M| (dense limit); |M| = 1; empty mid-region; all in one ragged batch."""
    from paper_2604_05438_amd import binding as B
    import parity_utils as PU
    w = I.WORKLOADS["l1b_32k"]
    A = w.n_sink + w.n_tail
    cases = [(1200, 0), (900, 900 - A), (900, 5000), (A + 1, 1), (A + 1, 0), (A, 3), (5, 2), (A + 300, 17)]
    layers = [I.make_layer(w, L=L, seq=i) for i, (L, _) in enumerate(cases)]
    ks = [k for _, k in cases]
    b = _batch(w, layers, ks)
    b.build()
    b.decode()
    assert b.status() == 0
    for i, ((L, k), P) in enumerate(zip(cases, layers)):
        rep = PU.check_layer(w, P, k, b, i, heads=[0, 5, 31])
        print("case", L, k, rep)
    # dense limit: with every mid token retrieved the output is full softmax attention
    from oracle import tkphi_oracle as orc
    O = PU.oracle_inputs(layers[1])
    y = b.result(1, "out")
    for g in (0, 13):
        ref = orc.full_attention(O["q"][g], O["K"][g // 4], O["V"][g // 4], w.score_scale)
        PU.check_output(y[g], ref, "dense limit")


SELECT_VARIANTS = {
    "spill": {"select_mode": 1},                            # every score written, plan / emit / resolve
    "direct": {"select_mode": 2},                           # short contexts: all scores in a row, one select kernel (longer: as filtered)
    "filtered": {"select_mode": 2, "scan_chunk": 1024},     # sampled bound, candidate lists (a chunk of its own rules the row out)
    "rescan": {"select_mode": 2, "select_test": 1},         # ... with a bound nothing passes: every head rescans
    "no_pruning": {"select_mode": 2, "select_test": 2},     # ... with a bound everything passes
}


@pytest.mark.parametrize("variant", list(SELECT_VARIANTS))
@pytest.mark.parametrize("shape,L,k", [("l3b_128k", 9000, 360), ("l1b_32k", 5000, 49), ("l1b_32k", 20011, 200)])
def test_select_pipelines(shape, L, k, variant):
    """The decode routes of the matrix-core shapes (spill; direct up to 12288 / 10240 mid tokens; filtered), and the filtered one's
    rare paths (threshold miss -> rescan of the head; no pruning -> every mid token a candidate), forced through
    tkphi_tuning at sizes the oracle checks in full; single problem, then a ragged batch with a tiny
    and an empty mid-region and budgets from 0 to most of the mid-region."""
    import parity_utils as PU
    tuning = SELECT_VARIANTS[variant]
    w = I.WORKLOADS[shape]
    rep, _, _ = _run_single(w, L, k, tuning=tuning)
    print("select", variant, shape, L, k, rep, flush=True)
    A = w.n_sink + w.n_tail
    Ls = [L // 2 + 3, 700, A + 2, A - 1, 2600, 1500]
    ks = [11, 5, 1, 3, 0, 1100]
    layers = [I.make_layer(w, L=l, seq=i) for i, l in enumerate(Ls)]
    b = _batch(w, layers, ks, tuning=tuning)
    b.build(); b.decode()
    from paper_2604_05438_amd import binding as B
    assert b.status() in (0, B.TKPHI_DEV_CLAMPED)      # (most of a mid-region retrieved: check_layer judges a clamp per head)
    for i, (P, kk) in enumerate(zip(layers, ks)):
        PU.check_layer(w, P, kk, b, i, heads=[0, w.n_q_heads // 2, w.n_q_heads - 1])


@pytest.mark.parametrize("variant", ["spill", "direct", "filtered"])
def test_graph_replay_matches_eager(variant):
    """A decode call captured into a HIP graph (it allocates nothing, synchronises nothing and records no
    memset) replayed several times, with eager decodes and synchronisations in between and the query changed
    between replays: every replay must reproduce the eager result bit for bit."""
    import torch
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS["l3b_128k"]
    Ls, ks = [6000, 2100], [240, 60]
    layers = [I.make_layer(w, L=l, seq=i) for i, l in enumerate(Ls)]
    b = _batch(w, layers, ks, tuning=SELECT_VARIANTS[variant])
    b.build(); b.decode()
    torch.cuda.synchronize()
    assert b.status() == 0
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr):
        b.decode()
    for rnd in range(4):
        for i, l in enumerate(Ls):                     # a new query for every problem, written in place
            q = H.to_device(I.make_layer(w, L=l, seq=i, query_index=rnd + 1, with_kv=False)["q"])
            b.dev[i]["q"].copy_(q)
        b.decode()
        torch.cuda.synchronize()
        eager = [b.result(i, "out").copy() for i in range(len(Ls))]
        for i in range(len(Ls)):
            b.dev[i]["out"].zero_()
        torch.cuda.synchronize()
        gr.replay()
        torch.cuda.synchronize()
        assert b.status() == 0
        for i in range(len(Ls)):
            assert np.array_equal(b.result(i, "out"), eager[i]), f"replay {rnd}, problem {i}"


@pytest.mark.parametrize("variant", list(SELECT_VARIANTS))
def test_exact_ties_take_lower_index(variant):
    """Duplicated keys give bit-equal scores on both sides: the index sets must match exactly."""
    from paper_2604_05438_amd import harness as H
    import parity_utils as PU
    tuning = SELECT_VARIANTS[variant]
    w = I.WORKLOADS["l1b_32k"]
    P = I.make_layer(w, L=3000)
    rng = np.random.default_rng(5)
    for h in range(w.n_kv_heads):
        src = rng.integers(w.n_sink, 3000 - w.n_tail, size=40)
        for s in src:                                  # 20 copies of each of 40 rows
            dst = rng.integers(w.n_sink, 3000 - w.n_tail, size=20)
            P["K"][h, dst] = P["K"][h, s]
    for k in (10, 29, 150):
        b = H.Batch(H.config_of(w, tuning=tuning), [P], [k], debug=True)
        b.build(); b.decode()
        rep = PU.check_layer(w, P, k, b, 0)
        print("ties", variant, k, rep)


@pytest.mark.parametrize("variant", ["filtered", "rescan", "no_pruning"])
@pytest.mark.parametrize("shape", ["l1b_32k", "l3b_128k"])
def test_batch_of_many_heads_uses_small_workgroups(shape, variant):
    """A batch with at least 512 query heads at head dimension 64 (16 problems x 32 heads) runs the fused select +
    gather kernel with 512-thread workgroups, two per CU; fewer heads, and head dimension 128 (22 problems x 24 heads
    here), run it with 1024 threads and one workgroup per head.  Same checks as for one problem: index sets, scores, outputs of several heads of every kind of problem against the
    oracle, through the common path, the rescan of every head and the path without pruning; one problem has identical
    keys (the radix passes), some have tiny budgets, one has no mid-region, one retrieves more than a gather round
    and more winners than stay in LDS."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    edge = w.n_sink + w.n_tail
    Ls = [5000, 2500, 777, 4229, 9000, edge + 1, edge, 40, 3001, 6000, 1500, 2048 + edge, 8192, 700, 12000, 4097]
    ks = [49, 24, 7, 300, 90, 1, 0, 3, 1, 600, 15, 20, 81, 700, 120, 40]
    if shape == "l3b_128k":
        Ls += [3000, 2000, 1000, 5000, 2500, 4000]
        ks += [30, 20, 10, 1400, 25, 40]
    layers = [I.make_layer(w, L=l, seq=i) for i, l in enumerate(Ls)]
    layers[8]["K"][:, :, :] = layers[8]["K"][:, 100:101, :]           # every score of problem 8 equal: Top-1 = first mid token
    tuning = dict(SELECT_VARIANTS[variant], scan_chunk=0)              # (a batch with 12000 tokens has lists at the default chunk)
    b = H.Batch(H.config_of(w, tuning=tuning), layers, ks, debug=True)
    assert w.n_q_heads * len(layers) >= 512
    b.build(); b.decode()
    assert b.status() == 0
    assert b.result(8, "topk_idx")[:, 0].tolist() == [w.n_sink] * w.n_q_heads
    for i in (0, 2, 3, 4, 5, 7, 9, 13, 14) + ((19,) if shape == "l3b_128k" else ()):
        rep = PU.check_layer(w, layers[i], ks[i], b, i, heads=[0, 13, w.n_q_heads - 1])
        print("many heads", shape, variant, "problem", i, Ls[i], ks[i], rep, flush=True)


@pytest.mark.parametrize("variant", list(SELECT_VARIANTS))
@pytest.mark.parametrize("shape,L", [("l1b_32k", 7000), ("l3b_128k", 3000), ("l1b_32k", 14000), ("l3b_128k", 12000)])
def test_all_scores_equal_slow_path(variant, shape, L):
    """Every key identical: the boundary bin holds the whole mid-region (more than the in-LDS candidate capacity), so the radix
    passes run; Top-K = first K.  7000 tokens at head dimension 64 and 3000 at 128 fit the array of packed candidates
    (12288, 10240): radix passes in LDS, also over the row of scores ("direct").  14000 and 12000 do not, and the
    boundary bin cannot be packed either: passes over the lists in global memory, of the score pass (filtered, no_pruning; the
    sampled bound equals every score) or of the rescan."""
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    P = I.make_layer(w, L=L)
    P["K"][:, :, :] = P["K"][:, 100:101, :]
    k = 61
    b = H.Batch(H.config_of(w, tuning=SELECT_VARIANTS[variant]), [P], [k], debug=True)
    b.build(); b.decode()
    idx = b.result(0, "topk_idx")
    for g in range(w.n_q_heads):
        assert idx[g, :k].tolist() == list(range(w.n_sink, w.n_sink + k))
    import parity_utils as PU
    rep = PU.check_layer(w, P, k, b, 0, heads=[0, 9])
    print("all-equal", rep)


@pytest.mark.parametrize("variant", ["filtered", "rescan", "no_pruning"])
def test_all_scores_equal_in_a_batch(variant):
    """The same in 512-thread workgroups (16 problems of 32 heads), whose packed array takes 4096 candidates: identical keys on
    5000 and 6100 tokens go through the lists in global memory, on 3000 through LDS."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS["l1b_32k"]
    Ls = [5000, 3000, 6100] + [700 + 50 * i for i in range(13)]
    ks = [49, 30, 700] + [7] * 13
    layers = [I.make_layer(w, L=l, seq=i) for i, l in enumerate(Ls)]
    for P in layers[:3]:
        P["K"][:, :, :] = P["K"][:, 100:101, :]
    b = H.Batch(H.config_of(w, tuning=SELECT_VARIANTS[variant]), layers, ks, debug=True)
    b.build(); b.decode()
    assert b.status() == 0
    for i in range(3):
        assert (b.result(i, "topk_idx")[:, :ks[i]] == np.arange(w.n_sink, w.n_sink + ks[i])).all()
    for i in (0, 1, 2, 3, 15):
        PU.check_layer(w, layers[i], ks[i], b, i, heads=[0, 13, 31])


@pytest.mark.parametrize("variant", ["spill", "direct", "filtered", "rescan", "no_pruning"])
@pytest.mark.parametrize("shape,L", [("l1b_32k", 3000), ("l3b_128k", 3000)])
def test_infinite_and_undefined_keys(variant, shape, L):
    """One infinite channel in some key rows of KV head 1, a row of NaN in KV head 2.  Scores of +infinity are retrieved first (by
    index), of -infinity never; selection-only outputs of the heads that see nothing but -infinity match an oracle that sees
    very negative scores in their place; the indices of KV head 2 are a valid set; every other head is as ever."""
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    w = I.WORKLOADS[shape]
    k, G = 30, w.group
    P = I.make_layer(w, L=L)
    q = I.to_f64(P["q"])
    c = int(np.argmin(np.abs(np.sign(q[G:2 * G]).sum(0))))             # a channel in which the group's queries have both signs
    Q = dict(P, K=P["K"].copy())                                       # the oracle's copy: 3e4 for infinity, the row of NaN as it was
    rows = np.array([w.n_sink, 77, 400, 401, 1999, L - w.n_tail - 1])
    P["K"][1, rows, c] = 0x7F80
    Q["K"][1, rows, c] = I.f32_to_bf16_bits(np.array([3e4], np.float32))[0]
    P["K"][2, 555, :] = 0x7FC0
    b = _batch(w, [P], [k], tuning=SELECT_VARIANTS[variant])
    b.build(); b.decode()
    S = [I.to_f64(x) for x in (b.result(0, "S"), b.result(0, "u"))]
    others = [g for g in range(w.n_q_heads) if g // G not in (1, 2)]
    assert all(np.isfinite(x[[h for h in range(w.n_kv_heads) if h not in (1, 2)]]).all() for x in S)
    res, S_or, u_or, _ = PU.oracle_layer(w, Q, k, heads=others[::5])
    PU.check_layer(w, Q, k, b, 0, heads=others[::5], summaries=(S_or, u_or))
    idx = b.result(0, "topk_idx")
    neg = []
    for g in range(G, 2 * G):
        got = idx[g, :k]
        assert (np.diff(got) > 0).all() and got[0] >= w.n_sink and got[-1] < L - w.n_tail
        assert np.isin(rows, got).all() if q[g, c] > 0 else not np.isin(rows, got).any(), (g, q[g, c])
        neg += [g] if q[g, c] < 0 else []
    for g in range(2 * G, 3 * G):
        got = idx[g, :k]
        assert (np.diff(got) > 0).all() and got[0] >= w.n_sink and got[-1] < L - w.n_tail
    assert neg
    b.decode(B.TKPHI_MODE_TOPK_ONLY)
    y = b.result(0, "out")
    for g, r in zip(neg, PU.oracle_layer(w, Q, k, heads=neg, S=S_or, u=u_or)[0]):
        PU.check_output(y[g], r["y_topk"], f"head {g} beside infinite keys")


def test_large_scores_use_the_max_shift():
    """Scores around +-60: unshifted exp would overflow fp32; the shifted path must agree
    with the float64 oracle."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_needles=0, n_outlier_channels=0, name="big", seed=99)
    P = I.make_layer(w, L=2000)
    q = I.to_f64(P["q"]) * 7.0
    P["q"] = I.f32_to_bf16_bits(q.astype(np.float32))
    b = H.Batch(H.config_of(w), [P], [19], debug=True)
    b.build(); b.decode()
    rep = PU.check_layer(w, P, 19, b, 0, heads=[0, 7, 20], check_aux=False)
    aux = b.result(0, "aux")
    assert np.abs(aux[:, 0]).max() > 20
    print("large", rep, "max shift", np.abs(aux[:, 0]).max())


def test_results_are_deterministic():
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS["l3b_128k"]
    P = I.make_layer(w, L=6000)
    b = H.Batch(H.config_of(w), [P], [59], debug=True)
    b.build()
    S0 = b.result(0, "S").copy()
    outs, idxs = [], []
    for _ in range(5):
        b.decode()
        outs.append(b.result(0, "out").copy())
        idxs.append(b.result(0, "topk_idx").copy())
    b.build()
    assert np.array_equal(S0, b.result(0, "S"))
    for o, ix in zip(outs[1:], idxs[1:]):
        assert np.array_equal(o, outs[0]) and np.array_equal(ix, idxs[0])


def test_bad_length_is_skipped_and_flagged():
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    import parity_utils as PU
    w = I.WORKLOADS["l1b_32k"]
    layers = [I.make_layer(w, L=1000, seq=0), I.make_layer(w, L=1500, seq=1)]
    b = H.Batch(H.config_of(w), layers, [9, 14], debug=True)
    # shrink the launch bound below the second problem's length (bypassing the host check)
    b.max_L = 1200
    b.ws_bytes = B.tkphi_workspace_bytes(b.cfg, b.n, 1500, b.max_K)
    b.dev[1]["out"].fill_(-7.0)
    b.dev[1]["S"].fill_(-3.0); b.dev[1]["u"].fill_(-3.0)
    b.ws.fill_(0xEE)                                   # the workspace need not be initialised
    b.build()
    assert b.status() == B.TKPHI_DEV_BAD_LENGTH        # the build records the skipped problem too ...
    assert (b.result(1, "S") == -3.0).all() and (b.result(1, "u") == -3.0).all()   # ... and leaves its S, u alone
    b.decode()
    assert b.status() & B.TKPHI_DEV_BAD_LENGTH
    assert (b.result(1, "out") == -7.0).all()
    rep = PU.check_layer(w, layers[0], 9, b, 0, heads=[0, 31])
    print("bad length", rep)


@pytest.mark.parametrize("d_emb", [0, 128])
def test_decode_replays_from_a_hip_graph(d_emb):
    """Both entry points only enqueue kernels on the caller's stream (with the MLP feature maps,
    d_emb > 0, also on the library's second stream, forked from and joined to the caller's): a
    captured decode step, replayed several times with eager work and synchronisations in between,
    reproduces the eager result bit for bit (and follows a changed query, since the table holds
    device pointers)."""
    import torch
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS["l3b_128k"]
    L, k = 6000, 59
    P = I.make_layer(w, L=L)
    if d_emb:
        P["mlp"] = I.make_mlp_phi(w, d_emb=d_emb)
    b = H.Batch(H.config_of(w, d_emb=d_emb), [P], [k], debug=True)
    b.build(); b.decode()
    torch.cuda.synchronize()
    y_eager = b.result(0, "out").copy()
    idx_eager = b.result(0, "topk_idx").copy()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        b.decode()                                   # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            b.decode()
    torch.cuda.synchronize()
    for rep in range(4):
        b.dev[0]["out"].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(b.result(0, "out"), y_eager), f"replay {rep} differs from the eager result"
        assert np.array_equal(b.result(0, "topk_idx"), idx_eager)
        # eager work between replays
        b.decode()
        torch.cuda.synchronize()
    # a new query through the same captured graph
    q2 = I.make_layer(w, L=L, query_index=5, with_kv=False)["q"]
    b.set_query(0, q2)
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    y_graph = b.result(0, "out").copy()
    b.decode()
    torch.cuda.synchronize()
    assert np.array_equal(b.result(0, "out"), y_graph)
    assert not np.array_equal(y_graph, y_eager)


def _check_diag(w, P, k, b, i, heads):
    import parity_utils as PU
    res, _, _, _ = PU.oracle_layer(w, P, k, heads=heads)
    dg = b.result(i, "diag")
    for g, r in zip(heads, res):
        row = dg[g].astype(np.float64)
        assert abs(row[0] - r["H_mid"]) <= 2e-4, f"head {g}: H_mid {row[0]} vs {r['H_mid']}"
        assert abs(row[1] - np.log(r["Z_M"])) <= 1e-4 * max(1.0, abs(np.log(r["Z_M"]))), f"head {g}: log Z_M"
        assert abs(row[2] - r["C_mid"]) <= 1e-4 * max(r["C_mid"], 1e-3), f"head {g}: C_mid {row[2]} vs {r['C_mid']}"
        assert abs(row[3] - r["rho_res"]) <= 5e-3 * max(r["rho_res"], 1e-6), f"head {g}: rho_res {row[3]} vs {r['rho_res']}"
        assert abs(row[4] - r["rho_res_star"]) <= 1e-4 * max(r["rho_res_star"], 1e-6), f"head {g}: rho_res*"
        if np.isfinite(r["log_Z_err"]):
            assert abs(row[5] - r["log_Z_err"]) <= 5e-3, f"head {g}: log error {row[5]} vs {r['log_Z_err']}"
        Z_A = r["Z_A"] + r["Z_G"]                      # generated tokens count with the exact anchors
        assert abs(row[6] - np.log(Z_A)) <= 1e-4 * max(1.0, abs(np.log(Z_A))), f"head {g}: log Z_A"


@pytest.mark.parametrize("shape,L,k,interleave", [("l3b_128k", 9000, 360, 0), ("l3b_128k", 20011, 200, 1),
                                                  ("l1b_32k", 5000, 0, 0), ("tiny_f32", 4096, 40, 0)])
def test_entropy_and_mass_diagnostics(shape, L, k, interleave):
    """The by-product diagnostics (normalised mid-region entropy, mid mass, Top-K mass recovery,
    residual shares, residual log-partition error) against the oracle; K = 0 included (nothing is
    retrieved but the score pass still runs); the output itself must not depend on the flag."""
    from paper_2604_05438_amd import binding as B
    import parity_utils as PU
    tuning = {"interleave": 1, "scan_chunk": 1024} if interleave else None
    w = I.WORKLOADS[shape]
    Ls = [L, max(L // 3, 100)]
    ks = [k, min(k, 7)]
    layers = [I.make_layer(w, L=l, seq=i) for i, l in enumerate(Ls)]
    b = _batch(w, layers, ks, tuning=tuning)
    b.build()
    b.decode(B.TKPHI_MODE_SUB)
    y_plain = [b.result(i, "out").copy() for i in range(2)]
    b.decode(B.TKPHI_MODE_SUB | B.TKPHI_FLAG_DIAG)
    assert b.status() == 0
    heads = sorted({0, w.n_q_heads // 2, w.n_q_heads - 1})
    for i, (P, kk) in enumerate(zip(layers, ks)):
        # (the diagnostics ride on the spill pipeline's passes; without the flag these shapes may take the
        # filtered pipeline, whose sums run in another order: equal to rounding, not bit for bit)
        y_d = b.result(i, "out")
        assert np.abs(y_d - y_plain[i]).max() <= 2e-5 * max(1.0, np.abs(y_plain[i]).max())
        PU.check_layer(w, P, kk, b, i, heads=heads)
        _check_diag(w, P, kk, b, i, heads)
    # within one pipeline the flag changes nothing at all
    b1 = _batch(w, layers, ks, tuning=dict(tuning or {}, select_mode=1))
    b1.build(); b1.decode(B.TKPHI_MODE_SUB)
    y1 = [b1.result(i, "out").copy() for i in range(2)]
    b1.decode(B.TKPHI_MODE_SUB | B.TKPHI_FLAG_DIAG)
    assert all(np.array_equal(b1.result(i, "out"), y1[i]) for i in range(2))


@pytest.mark.parametrize("shape,L,k", [("l3b_128k", 40000, 400), ("l1b_32k", 60000, 600), ("l3b_128k", 9000, 90)])
def test_diagnostics_of_one_problem_run_on_the_spill_chunks(shape, L, k):
    """A step with the diagnostics runs the spill pipeline; for one problem also in the spill pipeline's launch geometry, so that
    its output is that of a step forced through it bit for bit, whatever pipeline the plain step takes."""
    from paper_2604_05438_amd import binding as B
    w = I.WORKLOADS[shape]
    P = I.make_layer(w, L=L)
    y = []
    for tuning, flag in ((None, B.TKPHI_FLAG_DIAG), ({"select_mode": 1}, 0)):
        b = _batch(w, [P], [k], tuning=tuning)
        b.build(); b.decode(B.TKPHI_MODE_SUB | flag)
        assert b.status() == 0
        y.append(b.result(0, "out").copy())
        if flag:
            _check_diag(w, P, k, b, 0, [0, w.n_q_heads - 1])
    assert np.array_equal(y[0], y[1])


@pytest.mark.parametrize("shape,L,k", [("l3b_128k", 9000, 360), ("l1b_32k", 5000, 49), ("tiny_f32", 4096, 40),
                                       ("f32_gqa", 1500, 33)])
def test_cached_key_features(shape, L, k):
    """cfg.cache_features: the build also stores phi_k(k_i) of the mid-region, decode gathers the
    stored rows instead of recomputing them from the keys.  Same parity bar as the recomputing
    path, single problem and ragged batch; the cache itself against the oracle's features."""
    import parity_utils as PU
    from oracle import tkphi_oracle as orc
    if shape == "f32_gqa":
        w = dataclasses.replace(I.WORKLOADS["tiny_f32"], n_q_heads=4, n_kv_heads=2, d_head=128, d_phi=48,
                                name="f32_gqa", seed=77)
    else:
        w = I.WORKLOADS[shape]
    Ls = [L, L // 2 + 1, w.n_sink + w.n_tail + 1, 40]
    ks = [k, 9, 1, 3]
    layers = [I.make_layer(w, L=l, seq=i) for i, l in enumerate(Ls)]
    b = _batch(w, layers, ks, cache_features=True)
    b.build(); b.decode()
    assert b.status() == 0
    for i, (P, kk) in enumerate(zip(layers, ks)):
        PU.check_layer(w, P, kk, b, i, heads=sorted({0, w.n_q_heads // 2, w.n_q_heads - 1}))
    # the cache of problem 0, KV head 0, against the oracle's features (bf16 path: 16-bit values)
    O = PU.oracle_inputs(layers[0])
    _, M = orc.partition(Ls[0], w.n_sink, w.n_tail)
    F = orc.phi(O["K"][0, M], O["Wk"][0], O["bk"][0], w.phi_in_scale, w.phi_norm_coef)
    C = b.result(0, "phi_cache")[0].astype(np.float64)
    assert C.shape == F.shape
    rel = np.abs(C - F) / F
    assert rel.max() <= (2.0 ** -15 if w.dtype == "bf16" else 2e-5), f"cache rel err {rel.max():.3e}"


@pytest.mark.parametrize("cache", [True, False])
@pytest.mark.parametrize("shape,d_emb,L,k,mode", [("l3b_128k", 512, 9000, 360, ""), ("l1b_32k", 128, 10000, 49, ""),
                                                  ("bf16_wide_phi", 256, 1500, 33, ""), ("l1b_32k", 128, 10000, 49, "blocks"),
                                                  ("l3b_128k", 512, 4500, 45, "unfused")])
def test_mlp_feature_maps(shape, d_emb, L, k, mode, cache):
    """Learned feature maps (App. "Head-wise phi architecture"): the build evaluates the one-block
    ReZero MLP phi_k on the mid-region keys with the tiled matrix-core GEMM chain, stores the
    features and contracts them into S, u; decode evaluates phi_q per query head with the GEMV
    chain and gathers the stored key features.  Compared with the oracle run with phi_mlp on
    both sides: stored features, summaries, index sets, outputs; single problem and ragged batch
    (the 10000-token case crosses the 8192-token activation block).  The build runs as one
    persistent launch per problem by default; "blocks" forces the layer-wise launches per token block
    (residual + output fused), "unfused" all four layers apart (the path of widths that do not fuse).
    cache = False: no feature cache (Sec. "Retrieved-token subtraction": retrieved-key features recomputed at
    decode): the build keeps a group's features in the workspace, decode sends the retrieved rows through the chain."""
    import parity_utils as PU
    from oracle import tkphi_oracle as orc
    from paper_2604_05438_amd import harness as H
    if shape == "bf16_wide_phi":
        w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_q_heads=4, n_kv_heads=2, d_head=64, d_phi=192,
                                name="bf16_wide_phi", seed=78)
    else:
        w = I.WORKLOADS[shape]
    Ls = [L, L // 2 + 1, w.n_sink + w.n_tail + 1, 40]
    ks = [k, 9, 1, 3]
    layers = []
    for i, l in enumerate(Ls):
        P = I.make_layer(w, L=l, seq=i)
        P["mlp"] = I.make_mlp_phi(w, layer=i, d_emb=d_emb)
        layers.append(P)
    from paper_2604_05438_amd import binding as B
    b = H.Batch(H.config_of(w, d_emb=d_emb, cache_features=cache, tuning={"mlp_mode": B.MLP_MODES[mode]}), layers, ks, debug=True)
    b.build(); b.decode()
    assert b.status() == 0
    for i, (P, kk) in enumerate(zip(layers, ks)):
        rep = PU.check_layer(w, P, kk, b, i, heads=sorted({0, w.n_q_heads // 2, w.n_q_heads - 1}))
        print(f"mlp {shape} problem {i}: {rep}", flush=True)
    if cache:
        # stored features of problem 0 against the oracle's, every KV head
        O = PU.oracle_inputs(layers[0])
        _, fk = PU.mlp_feature_fns(layers[0])
        _, M = orc.partition(Ls[0], w.n_sink, w.n_tail)
        C = b.result(0, "phi_cache").astype(np.float64)
        worst = 0.0
        for h in range(w.n_kv_heads):
            F = fk[h](O["K"][h, M])
            assert C[h].shape == F.shape
            worst = max(worst, float((np.abs(C[h] - F) / F).max()))
        print(f"mlp {shape}: stored features, worst relative error {worst:.3e}", flush=True)
        assert worst <= PU.MLP_FEATURE_EPS
    # the other accounting modes and the diagnostics run on the same summaries
    from paper_2604_05438_amd import binding as B
    y_sub = b.result(0, "out").copy()
    b.decode(B.TKPHI_MODE_SUB | B.TKPHI_FLAG_DIAG)
    assert b.status() == 0
    assert np.array_equal(b.result(0, "out"), y_sub)
    _check_diag(w, layers[0], ks[0], b, 0, heads=[0, w.n_q_heads - 1])
    b.decode(B.TKPHI_MODE_NOSUB)
    PU.check_layer(w, layers[0], ks[0], b, 0, heads=[w.n_q_heads - 1], mode="nosub")


@pytest.mark.parametrize("shape,d_emb", [("l3b_128k", 0), ("l1b_32k", 0), ("tiny_f32", 0), ("l1b_32k", 128)])
def test_generated_tokens_stay_exact(shape, d_emb):
    """eq. (implemented_decode): rows [L, L + n_gen) of K, V are the generated-token prefix, exact
    and outside the prefill partition.  A ragged batch with n_gen = 0, 1, 64 (a whole extra tile),
    70 and the bound max_gen, one of them with an empty mid-region; every accounting mode; and the
    equivalence the oracle is pinned by: appending the generated tokens to the tail anchors of a
    longer prefill gives the same output."""
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    max_gen = 100
    A = w.n_sink + w.n_tail
    cases = [(3000, 29, 0), (2500, 24, 1), (1800, 18, 64), (2200, 0, 70), (2600, 40, max_gen), (A - 5, 3, 33)]
    layers = []
    for i, (L, k, ng) in enumerate(cases):
        P = I.make_layer(w, L=L + ng, seq=i)
        P["L"], P["n_gen"] = L, ng
        if d_emb:
            P["mlp"] = I.make_mlp_phi(w, layer=i, d_emb=d_emb)
        layers.append(P)
    ks = [k for _, k, _ in cases]
    b = H.Batch(H.config_of(w, d_emb=d_emb, max_gen=max_gen), layers, ks, debug=True)
    b.build()
    heads = sorted({0, w.n_q_heads // 2, w.n_q_heads - 1})
    for mode, flag in (("sub", B.TKPHI_MODE_SUB), ("nosub", B.TKPHI_MODE_NOSUB), ("topk", B.TKPHI_MODE_TOPK_ONLY)):
        b.decode(flag)
        assert b.status() == 0
        for i, (P, kk) in enumerate(zip(layers, ks)):
            rep = PU.check_layer(w, P, kk, b, i, heads=heads, mode=mode)
        print("generated tokens", shape, mode, rep, flush=True)
    b.decode(B.TKPHI_MODE_SUB | B.TKPHI_FLAG_DIAG)
    for i in (1, 4):
        _check_diag(w, layers[i], ks[i], b, i, heads=heads)
    # the same rows as a longer tail: n_tail' = n_tail + n_gen on a prefill of L + n_gen rows
    L, k, ng = cases[2]
    w2 = dataclasses.replace(w, n_tail=w.n_tail + ng)
    P2 = dict(layers[2]); P2["L"], P2["n_gen"] = L + ng, 0
    b2 = H.Batch(H.config_of(w2, d_emb=d_emb), [P2], [k], debug=True)
    b2.build(); b2.decode()
    b.decode()
    d1, d2 = b.result(2, "out").astype(np.float64), b2.result(0, "out").astype(np.float64)
    assert np.abs(d1 - d2).max() <= 2e-6 * max(1.0, np.abs(d2).max()), np.abs(d1 - d2).max()
    assert np.array_equal(b.result(2, "topk_idx")[:, :k], b2.result(0, "topk_idx")[:, :k])


@pytest.mark.parametrize("L,k", [(512, 1), (2000, 1), (512, 3), (4096, 7)])
def test_tied_needles_at_tiny_budgets(L, k):
    """The planted needles of the fp32 workload have the same score up to rounding (their
    float64 scores differ by ~1e-8): with fewer retrieved tokens than needles the fp32 kernels
    may keep another needle than the float64 oracle.  That is an admissible swap; the output is
    then compared with the oracle on the GPU's set, and the retrieved needles carry almost all
    of the attention mass, so a wrong weight or value row would show."""
    w = I.WORKLOADS["tiny_f32"]
    rep, b, P = _run_single(w, L, k)
    print("tied needles", L, k, rep)
    for mode in ("nosub", "topk"):
        _run_single(w, L, k, mode=mode)
