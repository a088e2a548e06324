"""The filtered score pass around its groups of rows (16 or 32), units (64 / 128 rows per wavefront, 256 / 512 per workgroup) and
chunks, which the pipelined loads run past at the end of every mid-region."""
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["l3b_128k", "l1b_32k"])
@pytest.mark.parametrize("chunk,interleave", [(0, 0), (512, 1), (1024, 2), (2048, 1)])
def test_score_groups_at_every_end(shape, chunk, interleave):
    """Every score (exported), index set and output of a ragged batch, filtered pipeline forced (with chunk 0 the pass of short
    contexts, which scores the same groups and stores all of them); scores to 1e-5, the bar of parity_utils.  The longest problem fills several chunks; budgets from one token to a fifth of the mid-region."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    mids = [1, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 255, 256, 257, 511, 513, 1023, 1025, 2049, 4500]
    ks = [max(1, m // (5 if i % 2 else 60)) for i, m in enumerate(mids)]
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i) for i, m in enumerate(mids)]
    b = H.Batch(H.config_of(w, tuning={"select_mode": 2, "scan_chunk": chunk, "interleave": interleave}), layers, ks, debug=True)
    b.build()
    b.decode()
    assert b.status() & ~2 == 0          # (the residual clamp may fire where nearly every mid token is retrieved)
    for i, (P, k) in enumerate(zip(layers, ks)):
        PU.check_layer(w, P, k, b, i, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


@pytest.mark.parametrize("shape", ["l3b_128k", "l1b_32k"])
def test_whole_line_loads_at_every_end(shape):
    """The layout of the key loads that calls of more than 64 MB of keys (by their bounds) take: mid-regions that end around the 8 rows
    of a load instruction, the 16 of a tile and the groups, far inside the bounds; one problem at a time (scores kept in LDS) and a
    batch (lists on the way).  Scores, index sets and outputs against the oracle."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    mids = [1, 7, 8, 9, 15, 16, 17, 24, 31, 33, 65, 127, 130, 1000, 2049]
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i) for i, m in enumerate(mids)]
    ks = [max(1, m // 9) for m in mids]
    for sel in ([1], [3], [6], [9], [14], range(len(mids))):
        b = H.Batch(H.config_of(w, tuning={"select_mode": 2}), [layers[i] for i in sel], [ks[i] for i in sel], debug=True, max_L=140000,
                    max_K=400)
        b.build()
        b.decode()
        assert b.status() & ~2 == 0
        for i, at in enumerate(sel):
            PU.check_layer(w, layers[at], ks[at], b, i, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


@pytest.mark.parametrize("shape", ["l3b_128k", "l1b_32k"])
@pytest.mark.parametrize("n_problems", [1, 7])
def test_scores_alike_in_both_layouts(shape, n_problems):
    """A call whose bounds allow for more than 64 MB of keys loads them in the other layout: its scores are those of the same problems under
    small bounds bit for bit, and no head of a sequence that is sampled whole (up to 1024 rows: its bound is its K-th score itself) loses
    a candidate to it.  A rescan would list every token: the workspace, cleared before the step, must not hold a head's worst one."""
    import numpy as np
    import torch
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    mids = [1000, 9, 1024, 300, 777, 1030, 5000][:n_problems]
    ks = [m // 60 + 1 for m in mids]
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i) for i, m in enumerate(mids)]
    res = []
    for max_L in (None, 140000):
        b = H.Batch(H.config_of(w, tuning={"select_mode": 2}), layers, ks, debug=True, max_L=max_L, max_K=400)
        b.build()
        b.ws.zero_()
        b.decode()
        assert b.status() & ~2 == 0
        res.append([{n: b.result(i, n) for n in ("scores", "topk_idx")} for i in range(n_problems)])
    words = b.ws[:b.ws_bytes // 8 * 8].view(torch.int64)
    for i, (small, large) in enumerate(zip(*res)):
        assert np.array_equal(small["scores"].view(np.uint32), large["scores"].view(np.uint32)), f"problem {i}: scores differ"
        assert np.array_equal(small["topk_idx"], large["topk_idx"])
        worst = large["scores"].argmin(1)
        bits = np.take_along_axis(large["scores"], worst[:, None], 1)[:, 0].view(np.uint32).astype(np.int64)
        listed = torch.isin(torch.from_numpy(worst.astype(np.int64) << 32 | bits).cuda(), words)
        assert not listed.any(), f"problem {i}: heads {listed.nonzero().flatten().tolist()} rescanned"


@pytest.mark.parametrize("shape", ["l3b_128k", "l1b_32k"])
@pytest.mark.parametrize("layout", ["token_major", "padded"])
def test_whole_line_loads_of_strided_and_undefined_keys(shape, layout):
    """Whole-line loads over rows that do not adjoin (all heads of a token in a row; rows padded by 16 bytes, so that most straddle cache
    lines), with an infinite channel in some rows of KV head 1 and a row of NaN in KV head 2: the scores of the plain layout over
    contiguous rows bit for bit (undefined ones where those are), the same index sets for the heads that see no NaN.  One problem and seven."""
    import numpy as np
    import torch
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    mids = [5000, 15, 1000, 1025, 64, 2050, 130]
    layers, strided = [], []
    for i, m in enumerate(mids):
        P = I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i)
        P["K"][1, [w.n_sink, w.n_sink + m // 2, w.n_sink + m - 1], 5 + 40 * (i % 2)] = 0x7F80
        P["K"][2, w.n_sink + m // 3, :] = 0x7FC0
        layers.append(P)
        dev = dict(P)
        for name in ("K", "V"):
            hm = H.to_device(P[name])
            if layout == "token_major":
                dev[name] = hm.permute(1, 0, 2).contiguous().permute(1, 0, 2)
            else:
                dev[name] = torch.zeros(*hm.shape[:2], w.d_head + 8, dtype=hm.dtype, device="cuda")[:, :, :w.d_head]
                dev[name].copy_(hm)
        strided.append(dev)
    plain = [g for g in range(w.n_q_heads) if g // w.group != 2]
    for n in (1, 7):
        res = []
        for inputs, max_L in ((layers, None), (strided, 140000)):
            b = H.Batch(H.config_of(w, tuning={"select_mode": 2}), inputs[:n], [m // 60 + 1 for m in mids[:n]], debug=True, max_L=max_L, max_K=400)
            b.build()
            b.decode()
            res.append([{x: b.result(i, x) for x in ("scores", "topk_idx")} for i in range(n)])
        for i, (want, got) in enumerate(zip(*res)):
            defined = ~np.isnan(want["scores"])
            assert np.array_equal(defined, ~np.isnan(got["scores"])) and not defined.all()
            assert np.array_equal(want["scores"][defined].view(np.uint32), got["scores"][defined].view(np.uint32)), f"problem {i}: scores differ"
            assert np.array_equal(want["topk_idx"][plain], got["topk_idx"][plain]), f"problem {i}: index sets differ"


@pytest.mark.parametrize("shape,L,k", [("l3b_128k", 2500, 200), ("l3b_128k", 40000, 400), ("l1b_32k", 20000, 300)])
def test_partials_of_several_workgroups(shape, L, k):
    """Several workgroups share a head and the last one merges what the others have handed it: steps of two queries in turn, without the
    export of the indices, on a workspace full of huge values, give the outputs of the steps with the export bit for bit (those against
    the oracle)."""
    import numpy as np
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    P = I.make_layer(w, L=L)
    queries = [P["q"], I.make_layer(w, L=L, seq=1)["q"]]
    want = []
    for debug in (True, False):
        b = H.Batch(H.config_of(w), [P], [k], debug=debug)
        b.build()
        for rep in range(2 if debug else 12):
            b.set_query(0, queries[rep % 2])
            b.ws.fill_(0x7f)             # (3.4e38 as a float)
            b.dev[0]["out"].zero_()
            b.decode()
            if debug:
                assert b.status() & ~2 == 0
                PU.check_layer(w, dict(P, q=queries[rep]), k, b, 0, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])
                want.append(b.result(0, "out"))
            else:
                assert np.array_equal(b.result(0, "out"), want[rep % 2]), f"step {rep} differs"


@pytest.mark.parametrize("shape,unit", [("l3b_128k", 64), ("l1b_32k", 128)])
@pytest.mark.parametrize("units,interleave", [(1, 0), (3, 1), (5, 2), (17, 1)])
def test_kept_scores_at_every_end(shape, unit, units, interleave):
    """One launch for the sample and the scores of one problem or a few: chunks of 1, 3, 5 and 17 units (a list is a quarter of a chunk:
    16 to 544 positions), mid-regions that end around units and
    chunks, and bounds of either sign (budgets beyond half of the mid-region).  Scores, index sets and outputs against the oracle."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    chunk = units * unit
    for mids in ([1], [unit - 1], [unit + 1], [chunk], [chunk + 1], [3 * chunk + unit // 2 + 1], [2500, 37, 2 * chunk - 1]):
        layers = [I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i) for i, m in enumerate(mids)]
        for share in (0.02, 0.6):
            ks = [max(1, int(m * share)) for m in mids]
            b = H.Batch(H.config_of(w, tuning={"select_mode": 2, "scan_chunk": chunk, "interleave": interleave}), layers, ks, debug=True)
            b.build()
            for _ in range(2):
                b.decode()
            assert b.status() & ~2 == 0  # (the residual clamp may fire where nearly every mid token is retrieved)
            for i, (P, k) in enumerate(zip(layers, ks)):
                PU.check_layer(w, P, k, b, i, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


@pytest.mark.parametrize("hq,hkv,d,chunk,max_L", [(8, 1, 128, 1024, 9000000), (4, 1, 64, 256, 700000), (8, 1, 128, 1024, 2000000)])
def test_given_chunk_too_short_for_the_bounds(hq, hkv, d, chunk, max_L):
    """A given chunk grows until 2048 of them hold the bounds: where its scores then pass what a workgroup can keep in LDS (the first case)
    the call takes the pass that does not keep them."""
    import dataclasses
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l3b_128k" if d == 128 else "l1b_32k"], n_q_heads=hq, n_kv_heads=hkv)
    P = I.make_layer(w, L=3000)
    b = H.Batch(H.config_of(w, tuning={"select_mode": 2, "scan_chunk": chunk}), [P], [40], debug=True, max_L=max_L, max_K=400)
    b.build()
    b.decode()
    assert b.status() & ~2 == 0
    PU.check_layer(w, P, 40, b, 0)


def _kernel_attributes(name, more=""):
    import ctypes
    from paper_2604_05438_amd import binding as B

    class Attributes(ctypes.Structure):                     # hipFuncAttributes
        _fields_ = [("binaryVersion", ctypes.c_int), ("cacheModeCA", ctypes.c_int), ("constSizeBytes", ctypes.c_size_t),
                    ("localSizeBytes", ctypes.c_size_t), ("maxDynamicSharedSizeBytes", ctypes.c_int), ("maxThreadsPerBlock", ctypes.c_int),
                    ("numRegs", ctypes.c_int), ("preferredShmemCarveout", ctypes.c_int), ("ptxVersion", ctypes.c_int),
                    ("sharedSizeBytes", ctypes.c_size_t)]

    attr = Attributes()
    kernel = ctypes.c_void_p.in_dll(B.lib(), f"_ZN5tkphi{name}EvNS_4GeomEPK13tkphi_problemPc{more}")
    assert B.lib().hipFuncGetAttributes(ctypes.byref(attr), ctypes.byref(kernel)) == 0
    return attr


@pytest.mark.parametrize("d,tiles", [(64, 8), (128, 4)])
@pytest.mark.parametrize("stream", [0, 1])
@pytest.mark.parametrize("name,more", [("18score_fused_kernel", ""), ("22score_fused_few_kernel", "NS_9FusedJobsE")])
def test_kept_scores_leave_room_for_two_workgroups(d, tiles, stream, name, more):
    """The one-launch score pass keeps up to 79872 bytes of scores per workgroup so that two share the 160 KB of a CU: what its kernel
    holds besides must fit the 2 KB left of each half."""
    assert _kernel_attributes(f"{name}ILi{d}ELi{tiles}ELb{stream}EE", more).sharedSizeBytes <= 81920 - 79872


@pytest.mark.parametrize("name,wavefronts", [("18decode_side_kernelILi64EE", 7), ("18decode_side_kernelILi128EE", 7),
                                             ("19score_direct_kernelILi64ELi8ELi0EE", 5), ("19score_direct_kernelILi128ELi4ELi0EE", 6)])
def test_batch_jobs_keep_their_wavefronts(name, wavefronts):
    """The launches that carry the phi and anchor jobs of batches are throughput work: the wavefronts per SIMD that they were measured with
    (512 registers, dealt in eights)."""
    assert 0 < _kernel_attributes(name).numRegs <= 512 // wavefronts // 8 * 8


@pytest.mark.parametrize("shape,n_mid,k,select_test", [
    ("l3b_128k", 11000, 100, 0), ("l1b_32k", 13000, 700, 0),      # a hot stretch overflows the compact heads of its lists: several sweeps
    ("l3b_128k", 9000, 100, 0), ("l1b_32k", 9000, 700, 0),        # short contexts: no lists, the row of scores is packed as it is
    ("l3b_128k", 13000, 400, 2), ("l1b_32k", 14000, 1500, 2),     # every token a candidate, more than the packed array: boundary bin first
    ("l1b_32k", 14000, 13500, 2),                                 # a budget beyond the packed array: every phase from the lists
    ("l3b_128k", 13000, 900, 1), ("l1b_32k", 14000, 300, 1)])     # no bound for half of the chunks, and nothing passes that of the others: rescan, then as above
def test_candidate_packing(shape, n_mid, k, select_test):
    """The select kernel's ways of bringing the candidates of a head together, where neighbouring tokens score alike (rows
    [2000, 2400) lean towards a query of their group, so their lists hold far more than the expected share).  One problem
    (several workgroups per head share the packed array) and a batch of three (one each), against the oracle."""
    import numpy as np
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    layers = []
    for i, m in enumerate((n_mid, n_mid // 2 + 5, 700)):
        P = I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i)
        if m > 2400:
            K, q = I.bf16_bits_to_f32(P["K"]), I.bf16_bits_to_f32(P["q"])
            for h in range(w.n_kv_heads):
                lean = q[h * w.group + h % w.group]
                K[h, 2000:2400] = 0.6 * K[h, 2000:2400] + np.float32(0.35) * lean
            P["K"] = I.f32_to_bf16_bits(K)
        layers.append(P)
    ks = [k, max(1, k // 3), min(k, 650) // 7]
    for n in (1, 3):
        b = H.Batch(H.config_of(w, tuning={"select_mode": 2, "select_test": select_test}), layers[:n], ks[:n], debug=True)
        b.build()
        b.decode()
        assert b.status() & ~2 == 0      # (the residual clamp may fire where nearly every mid token is retrieved)
        for i in range(n):
            PU.check_layer(w, layers[i], ks[i], b, i, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


@pytest.mark.parametrize("shape,max_mid", [("l1b_32k", 12288), ("l1b_32k", 12289), ("l3b_128k", 10240), ("l3b_128k", 10241), ("l1b_32k", 4096)])
@pytest.mark.parametrize("n_problems", [1, 2, 18])
def test_short_contexts(shape, max_mid, n_problems):
    """Contexts whose scores the select kernel takes as a whole (no sampled bound, one launch less): the largest mid-region
    of that path and one token more, one problem, two, and a batch whose heads take the 512-thread select (limit 4096); lengths
    down to one token, budgets from one token to the largest of the filtered pipeline, generated tokens, ties."""
    import numpy as np
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    max_gen = 70
    mids = ([max_mid, 1, 63, 64, 65, 255, 257, 511, 513, 700, 1023, 1500] * 2)[:n_problems]
    ks = [max(1, m // (12 if i % 2 == 0 else 90)) for i, m in enumerate(mids)]
    layers = []
    for i, m in enumerate(mids):
        gen = (i * 37 + 3) % (max_gen + 1)
        P = I.make_layer(w, L=w.n_sink + w.n_tail + m + gen, seq=i)
        P["L"], P["n_gen"] = w.n_sink + w.n_tail + m, gen
        if i == 0:                       # equal rows: ties across the whole region, taken by lower index
            P["K"][:, 100:900] = P["K"][:, 100:101]
        layers.append(P)
    b = H.Batch(H.config_of(w, max_gen=max_gen), layers, ks, debug=True)
    b.build()
    b.decode()
    assert b.status() & ~2 == 0          # (the residual clamp may fire where nearly every mid token is retrieved)
    for i, (P, k) in enumerate(zip(layers, ks)):
        PU.check_layer(w, P, k, b, i, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


@pytest.mark.parametrize("shape,big_L,big_K,calls", [
    # shorter sequences and smaller budgets than the workspace was sized for: other chunks, one-launch selection, other pipeline
    ("l3b_128k", 65536, 655, [(50000, 500), (50000, 3000), (12000, 120), (10308, 100), (300, 20)]),
    ("l1b_32k", 65536, 1310, [(65536, 1000), (50000, 1000), (40000, 320), (13000, 1000), (12356, 123), (700, 600)]),
    ("l1b_32k", 40000, 20000, [(40000, 700), (40000, 3000), (39000, 3900)])])
@pytest.mark.parametrize("exact", [False, True])
def test_workspace_sized_for_larger_bounds(shape, big_L, big_K, calls, exact):
    """A workspace sized for a call's largest bounds serves the smaller ones, with its own size (exact) or more than that, and
    an index set and output that match the oracle; what the call itself reports as needed is enough as well."""
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    for L, k in calls:
        P = I.make_layer(w, L=L, seq=0)
        k = min(k, big_K)
        b = H.Batch(H.config_of(w), [P], [k], debug=True)
        if not exact:
            b.ws_bytes = B.tkphi_workspace_bytes(b.cfg, 1, big_L, big_K)
            b.ws = B.alloc_workspace(b.ws_bytes, "cuda")
        b.build()
        b.decode()
        assert b.status() & ~2 == 0
        PU.check_layer(w, P, k, b, 0, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


@pytest.mark.parametrize("shape,L,k", [("l1b_32k", 60000, 1200), ("l1b_32k", 60000, 4500), ("l3b_128k", 50000, 1500), ("l1b_32k", 30000, 300)])
def test_static_scratch_budgets(shape, L, k):
    """Budgets of 2 to 7.5 % whose faster pipeline needs more than the 32 MiB of static scratch run with the smaller one."""
    import torch
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    P = I.make_layer(w, L=L, seq=0)
    b = H.Batch(H.config_of(w), [P], [k], debug=True)
    b.build()
    B.tkphi_decode_static(b.cfg, b.table.data_ptr(), 1, b.max_L, b.max_K, 0, B.current_stream_ptr())
    torch.cuda.synchronize()
    PU.check_layer(w, P, k, b, 0, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


def test_static_scratch_holds_the_two_launch_pass():
    """16 heads over 2 KV heads, 109000 tokens: the chunks of the one-launch score pass need more than the 32 MiB of static scratch, those of
    the pass with a launch for the sample fit."""
    import dataclasses
    import torch
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l1b_32k"], n_q_heads=16, n_kv_heads=2)
    P = I.make_layer(w, L=109000)
    b = H.Batch(H.config_of(w), [P], [270], debug=True)
    b.build()
    B.tkphi_decode_static(b.cfg, b.table.data_ptr(), 1, b.max_L, b.max_K, 0, B.current_stream_ptr())
    torch.cuda.synchronize()
    PU.check_layer(w, P, 270, b, 0, heads=[0, 7, 15])


def test_diagnostics_in_a_workspace_sized_for_a_larger_budget():
    """A step with the diagnostics takes other chunks than one without: a workspace sized for a budget of 2 % serves one of 5 tokens."""
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS["l1b_32k"]
    layers = [I.make_layer(w, L=L, seq=i) for i, L in enumerate((13753, 9000))]
    b = H.Batch(H.config_of(w), layers, [5, 5], debug=True)
    b.ws_bytes = B.tkphi_workspace_bytes(b.cfg, 2, 13753, 275)
    b.ws = B.alloc_workspace(b.ws_bytes, "cuda")
    b.build()
    b.decode(B.TKPHI_MODE_SUB | B.TKPHI_FLAG_DIAG)
    assert b.status() & ~2 == 0
    for i, P in enumerate(layers):
        PU.check_layer(w, P, 5, b, i, heads=[0, 17, 31])


@pytest.mark.parametrize("shape,L,k,n", [("l3b_128k", 14000, 139, 1), ("l1b_32k", 5000, 49, 1), ("l3b_128k", 14000, 139, 5)])
def test_each_decode_route_replays_from_a_hip_graph(shape, L, k, n):
    """The sampled-bound route of one problem (two launches; the bounds handed over inside the first) and of a batch of 40 KV heads (three),
    and the short-context one (two), captured and replayed with eager work between."""
    import numpy as np
    import torch
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    b = H.Batch(H.config_of(w), [I.make_layer(w, L=L, seq=i) for i in range(n)], [k] * n, debug=True)
    b.build(); b.decode()
    torch.cuda.synchronize()
    eager = {(i, x): b.result(i, x).copy() for i in range(n) for x in ("out", "topk_idx")}
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        b.decode()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            b.decode()
    torch.cuda.synchronize()
    for rep in range(3):
        for dev in b.dev:
            dev["out"].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for (i, x), y in eager.items():
            assert np.array_equal(b.result(i, x), y), f"replay {rep}: {x} of problem {i} differs from the eager result"
        b.decode()
        torch.cuda.synchronize()


@pytest.mark.parametrize("hq,hkv,d,n,max_mid,max_K,filtered", [
    (24, 8, 128, 1, 131004, 1310, True), (24, 8, 128, 1, 131004, 7800, True), (24, 8, 128, 1, 131004, 10400, False),     # winners beyond the packed array
    (3, 1, 128, 1, 131004, 1310, True), (3, 1, 128, 1, 131004, 5240, False), (3, 1, 128, 1, 32000, 2040, True),          # few heads
    (4, 1, 64, 1, 12000, 1000, True), (4, 1, 64, 1, 12000, 1001, False),                                                 # short context, 1/12
    (32, 8, 64, 18, 40000, 1600, True), (32, 8, 64, 18, 40000, 3200, False),                                             # 576 heads: 3/4 of three rounds
    (24, 8, 128, 11, 16000, 250, True), (24, 8, 128, 11, 16000, 320, False)])                                            # 264 heads: second round empty
def test_pipeline_by_bounds(hq, hkv, d, n, max_mid, max_K, filtered):
    """Which pipeline a call takes follows from its bounds (the problems themselves are short here): the stages that ran say it;
    either way the result is the oracle's."""
    import dataclasses
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l3b_128k" if d == 128 else "l1b_32k"], n_q_heads=hq, n_kv_heads=hkv)
    layers = [I.make_layer(w, L=700 + 13 * i, seq=i) for i in range(n)]
    b = H.Batch(H.config_of(w), layers, [40] * n, debug=True, max_L=max_mid + w.n_sink + w.n_tail, max_K=max_K)
    b.build()
    stages = dict(zip(B.STAGES, b.decode_stage_times()))
    assert (stages["select"] > 0) == filtered and (stages["merge"] > 0) == (not filtered), stages
    for i in (0, n - 1):
        PU.check_layer(w, layers[i], 40, b, i, heads=[0, hq - 1])


@pytest.mark.parametrize("shape,n_mid,n_problems", [("l1b_32k", 14000, 1), ("l1b_32k", 14000, 9), ("l1b_32k", 5000, 17), ("l3b_128k", 11000, 1), ("l3b_128k", 11000, 11)])
def test_sampled_rows_above_all_others(shape, n_mid, n_problems):
    """The rows that the bound is sampled from lean towards one query of their group, so that its K best are among them and the
    bound lies above its K-th score: that head misses and rescans, its neighbours, scanned in the same pass, do not.  One
    problem (several workgroups per head, which write a second set of lists) and batches (one each, which writes its lists
    over; 512 threads from 512 heads on): index sets, scores and outputs against the oracle."""
    import numpy as np
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    layers, k = [], n_mid // 100
    m = min(1024, max(512, n_mid // 64)) // 16 * 16                     # the sample: groups of 16 rows at equal distances
    rows = np.array([(s >> 4) * (n_mid // (m >> 4)) + (s & 15) for s in range(m)]) + w.n_sink
    for i in range(n_problems):
        P = I.make_layer(w, L=w.n_sink + w.n_tail + n_mid, seq=i % 3)
        K, q = I.bf16_bits_to_f32(P["K"]), I.bf16_bits_to_f32(P["q"])
        h, g = i % w.n_kv_heads, i % w.group
        K[h, rows] = 0.5 * K[h, rows] + np.float32(0.6) * q[h * w.group + g]
        P["K"] = I.f32_to_bf16_bits(K)
        layers.append(P)
    b = H.Batch(H.config_of(w, tuning={"select_mode": 2, "scan_chunk": 1024}), layers, [k] * n_problems, debug=True)
    b.build()
    for _ in range(2):
        b.decode()
    assert b.status() & ~2 == 0
    for i in sorted({0, 1 % n_problems, n_problems - 1}):
        hot = (i % w.n_kv_heads) * w.group + i % w.group
        PU.check_layer(w, layers[i], k, b, i, heads=sorted({hot, hot ^ 1, (hot + w.group) % w.n_q_heads}))
        assert np.isin(b.result(i, "topk_idx")[hot, :k], rows).mean() > 0.9        # (the case is what it says: the bound misses)


@pytest.mark.parametrize("hq,hkv,d", [(8, 1, 64), (16, 2, 128)])
def test_contexts_beyond_the_kept_chunks(hq, hkv, d):
    """A single sequence of more than 128 chunks of kept scores per KV head: sample and score pass as two launches, heads against the oracle."""
    import dataclasses
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l3b_128k" if d == 128 else "l1b_32k"], n_q_heads=hq, n_kv_heads=hkv)
    P = I.make_layer(w, L=321000)
    b = H.Batch(H.config_of(w), [P], [900], debug=True)
    b.build()
    stages = dict(zip(B.STAGES, b.decode_stage_times()))
    assert stages["prep"] > 0 and stages["select"] > 0 and b.status() == 0
    PU.check_layer(w, P, 900, b, 0, heads=[0, hq - 1])


@pytest.mark.parametrize("shape,chunk,max_L", [("l3b_128k", 64, None), ("l3b_128k", 320, None), ("l3b_128k", 0, 140000), ("l1b_32k", 128, None),
                                               ("l1b_32k", 1280, None), ("l1b_32k", 0, 140000)])
def test_rescan_at_every_list_length(shape, chunk, max_L):
    """A head that lists its keys again, in lists of 16 tokens to more than it has, mid-regions around tiles and lists: one problem (a second
    set of lists) and seven (more than 128 heads: the first set over), against the oracle."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = I.WORKLOADS[shape]
    mids = [1000, 1, 15, 17, 64, 1281, 2500]
    ks = [max(1, m // 12) for m in mids]
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + m, seq=i) for i, m in enumerate(mids)]
    for sel in ([0], [3], [5], range(7)):
        b = H.Batch(H.config_of(w, tuning={"select_mode": 2, "select_test": 1, "scan_chunk": chunk}), [layers[i] for i in sel], [ks[i] for i in sel],
                    debug=True, max_L=max_L, max_K=400)
        b.build()
        b.decode()
        assert b.status() & ~2 == 0
        for i, at in enumerate(sel):
            PU.check_layer(w, layers[at], ks[at], b, i, heads=[0, w.n_q_heads // 2 + 1, w.n_q_heads - 1])


@pytest.mark.parametrize("hq,hkv,d,L,k", [(3, 1, 128, 70000, 700), (8, 1, 64, 70000, 1500), (1, 1, 128, 20000, 100), (4, 2, 64, 50000, 400)])
def test_few_kv_heads(hq, hkv, d, L, k):
    """One or two KV heads over a long context: at most 128 chunks per head, fewer workgroups than CUs.  All heads against the
    oracle, at the library's own geometry."""
    import dataclasses
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = dataclasses.replace(I.WORKLOADS["l3b_128k" if d == 128 else "l1b_32k"], n_q_heads=hq, n_kv_heads=hkv)
    P = I.make_layer(w, L=L)
    b = H.Batch(H.config_of(w), [P], [k], debug=True)
    b.build()
    b.decode()
    assert b.status() == 0
    PU.check_layer(w, P, k, b, 0)
