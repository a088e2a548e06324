"""The gather and merge launches of the spill pipeline: the summary terms beside the gather, in every kernel and accounting mode."""
import dataclasses

import numpy as np
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


def _workload(dtype, d, dphi, seed):
    return dataclasses.replace(I.WORKLOADS["tiny_f32"], dtype=dtype, n_q_heads=8, n_kv_heads=2, d_head=d, d_phi=dphi, seed=seed)


@pytest.mark.parametrize("dtype,d,dphi,cache", [("bf16", 64, 64, False), ("bf16", 128, 128, False), ("bf16", 128, 48, False), ("f32", 64, 64, False),
                                                ("bf16", 64, 64, True), ("f32", 128, 16, True)])
def test_summaries_stay_untouched_where_nothing_reads_them(dtype, d, dphi, cache):
    """Without a residual branch (selection only; every mid token retrieved and subtracted) the spill pipeline reads neither S nor u: with both
    pointers null it gives what it gave with them, bit for bit."""
    import torch
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = _workload(dtype, d, dphi, 101)
    mid = 300
    layers = [I.make_layer(w, L=w.n_sink + w.n_tail + mid, seq=i) for i in range(2)]
    for mode, ks in ((B.TKPHI_MODE_TOPK_ONLY, [20, mid]), (B.TKPHI_MODE_SUB, [mid, mid])):
        b = H.Batch(H.config_of(w, cache_features=cache, tuning={"select_mode": 1}), layers, ks)
        b.build()
        b.decode(mode)
        want = [b.result(i, "out") for i in range(2)]
        for i in range(2):
            b.host_table[i].S = None
            b.host_table[i].u = None
            b.dev[i]["out"].zero_()
            assert np.isfinite(want[i]).all()
        b.set_topk(0, ks[0])                            # (uploads the table)
        b.decode(mode)
        torch.cuda.synchronize()
        assert b.status() == 0
        for i in range(2):
            assert np.array_equal(b.result(i, "out"), want[i])
