"""The score launch of batches: chunks of all KV heads, behind them the phi and anchor jobs, in one numbering."""
import dataclasses

import numpy as np
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


def _workload(d, hq, hkv, tail=64):
    return dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype="bf16", n_q_heads=hq, n_kv_heads=hkv, d_head=d, d_phi=d, n_tail=tail, seed=103)


@pytest.mark.parametrize("d,hq,hkv,chunk,max_gen", [(64, 8, 8, 512, 0), (64, 32, 4, 0, 70), (64, 6, 2, 512, 3), (128, 9, 3, 0, 0), (128, 8, 1, 256, 130),
                                                    (128, 4, 4, 256, 0)])
def test_ragged_batches(d, hq, hkv, chunk, max_gen):
    """Ragged problems, one of them without a mid-region and one that is skipped, from 1 to 80 chunks per KV head, against the oracle."""
    import parity_utils as PU
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = _workload(d, hq, hkv)
    n = max(12, 40 // hkv + 1)                          # (beyond 32 KV heads: two launches)
    lens = [20001, 14000, 8300, 4097, 1500, 700, 68, 40, 20001, 14000, 1500, 69]
    ks = [150, 30, 80, 17, 3, 60, 0, 0, 0, 200, 1, 1]
    small = {}
    layers, kk = [], []
    for i in range(n):
        L, k = lens[i % 12], ks[i % 12]
        if L not in small:
            gen = max_gen if L % 2 else max_gen // 2
            small[L] = I.make_layer(w, L=L + gen, seq=len(small))
            small[L].update(L=L, n_gen=gen)
        layers.append(small[L])
        kk.append(k)
    tuning = {"scan_chunk": chunk, "select_mode": 2}
    b = H.Batch(H.config_of(w, tuning=tuning, max_gen=max_gen), layers, kk, debug=True)
    b.build()
    b.host_table[4].L = b.max_L + 1                     # skipped (at decode only)
    b.dev[4]["out"].fill_(7.0)
    b.set_topk(0, kk[0])                                # (uploads the table)
    for _ in range(2):
        b.decode()
    assert b.status() & ~2 == B.TKPHI_DEV_BAD_LENGTH
    assert (b.result(4, "out") == 7.0).all()
    seen = set()
    for i, (P, k) in enumerate(zip(layers, kk)):
        if i == 4 or (int(P["L"]), k) in seen:
            continue
        seen.add((int(P["L"]), k))
        PU.check_layer(w, P, k, b, i, heads=[0, hq - 1], sum_tol=2e-5)


@pytest.mark.parametrize("n", [1, 3, 40])
@pytest.mark.parametrize("d", [64, 128])
def test_no_mid_region_at_all(d, n):
    """Bounds without a mid-region on the candidate-list route (a given chunk keeps the short-context row away): dense attention over all tokens."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = _workload(d, 4, 2)
    layers = [I.make_layer(w, L=60 + i % 9, seq=i % 9) for i in range(n)]
    b = H.Batch(H.config_of(w, tuning={"scan_chunk": 512}), layers, [0] * n, debug=True)
    b.build()
    b.decode()
    assert b.status() == 0
    for i in range(min(n, 9)):
        PU.check_layer(w, layers[i], 0, b, i, sum_tol=2e-5)


def test_one_problem_of_many_jobs():
    """More phi and anchor jobs than the prep launch takes beside the sample (generated tokens of 40 anchor tiles for 32 heads)."""
    import parity_utils as PU
    from paper_2604_05438_amd import harness as H
    w = _workload(64, 32, 8)
    gen = 40 * 64 - 68
    P = I.make_layer(w, L=9000 + gen)
    P.update(L=9000, n_gen=gen)
    b = H.Batch(H.config_of(w, tuning={"scan_chunk": 512, "select_mode": 2, "select_test": 2}, max_gen=gen), [P], [50], debug=True)
    b.build()
    b.decode()
    assert b.status() & ~2 == 0
    PU.check_layer(w, P, 50, b, 0, heads=[0, 17, 31], sum_tol=2e-5)


def test_grid_of_two_rows():
    """65535 problems of 4 heads: 1.6 million workgroups.  All problems are the same one, and so are their outputs."""
    import ctypes as C

    import torch
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = _workload(64, 4, 4)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 1300)
    n, k = 65535, 13
    one = H.Batch(H.config_of(w, tuning={"scan_chunk": 512, "select_mode": 2}), [P], [k])
    one.build()
    out = torch.full((n, 4, 64), float("nan"), device="cuda")
    rec = np.frombuffer(bytes(memoryview(one.host_table).cast("B")), dtype=np.uint8)
    table = np.tile(rec, (n, 1))
    at = B.tkphi_problem.out.offset
    table[:, at:at + 8] = (out.data_ptr() + np.arange(n, dtype=np.uint64) * (4 * 64 * 4)).reshape(n, 1).view(np.uint8)
    dev = torch.from_numpy(table.reshape(-1)).cuda()
    size = B.tkphi_workspace_bytes(one.cfg, n, one.max_L, k)
    ws = B.alloc_workspace(size)
    assert C.sizeof(B.tkphi_problem) == rec.size
    B.tkphi_decode(one.cfg, dev.data_ptr(), n, one.max_L, k, B.TKPHI_MODE_SUB, ws.data_ptr(), size, B.current_stream_ptr())
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out[0]).all()) and bool((out == out[0]).all())
    one.decode()
    assert float((out[0] - one.dev[0]["out"]).abs().max()) <= 1e-5      # (other splits of the same sums: fp32 rounding of values below 1)
