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


def _fma32(a, b, x):
    from fractions import Fraction
    return np.float32(float(Fraction(float(a)) * Fraction(float(b)) + Fraction(float(x))))


@pytest.mark.parametrize("dtype,d,dphi,cache", [("bf16", 64, 64, False), ("bf16", 128, 128, False), ("bf16", 128, 16, False), ("bf16", 64, 256, False),
                                                ("bf16", 64, 64, True), ("f32", 128, 256, False), ("f32", 64, 48, True)])
def test_summary_terms(dtype, d, dphi, cache):
    """phi_q . u_M is a chain of fused multiply-adds in feature order, bit for bit; S_M^T phi_q against 64 bits.  phi_q itself is read off
    the residual sums of S = shifted identities.  NOSUB: the residual terms of `aux` are then those of S and u alone."""
    import torch
    from paper_2604_05438_amd import binding as B
    from paper_2604_05438_amd import harness as H
    w = _workload(dtype, d, dphi, 102)
    P = I.make_layer(w, L=w.n_sink + w.n_tail + 300)
    b = H.Batch(H.config_of(w, cache_features=cache, tuning={"select_mode": 1}), [P], [20], debug=True)
    b.build()
    S, u = b.dev[0]["S"], b.dev[0]["u"]
    rng = np.random.default_rng(5)
    u_np = np.exp(rng.standard_normal((w.n_kv_heads, dphi))).astype(np.float32)
    u.copy_(torch.from_numpy(u_np))
    phi_q = np.zeros((w.n_q_heads, dphi), np.float32)
    for k in range(0, dphi, d):
        S.zero_()
        for j in range(k, min(k + d, dphi)):
            S[:, j, j - k] = 1.0
        b.decode(B.TKPHI_MODE_NOSUB)
        n = min(d, dphi - k)
        phi_q[:, k:k + n] = b.result(0, "aux")[:, 4 + d:4 + d + n]
    assert (phi_q > 0).all()
    aux, rounded_differs = b.result(0, "aux"), False
    for h in range(w.n_q_heads):
        x = np.float32(0.0)
        r = np.float32(0.0)
        for j in range(dphi):
            uj = u_np[h // (w.n_q_heads // w.n_kv_heads), j]
            x = _fma32(phi_q[h, j], uj, x)
            r = np.float32(r + np.float32(phi_q[h, j] * uj))
        assert aux[h, 2] == x, (h, aux[h, 2], x)
        rounded_differs |= bool(x != r)
    assert rounded_differs                              # (products rounded on the way would show)
    S_np = rng.standard_normal((w.n_kv_heads, dphi, d)).astype(np.float32)
    S.copy_(torch.from_numpy(S_np))
    b.decode(B.TKPHI_MODE_NOSUB)
    aux = b.result(0, "aux")
    for h in range(w.n_q_heads):
        terms = phi_q[h].astype(np.float64)[:, None] * S_np[h // (w.n_q_heads // w.n_kv_heads)].astype(np.float64)
        # dphi fused multiply-adds and sums, each within 2^-24 of sums no larger than the sum of the terms' sizes
        assert (np.abs(aux[h, 4 + d:4 + 2 * d] - terms.sum(0)) <= (dphi + 16) * 2.0 ** -24 * np.abs(terms).sum(0)).all()
