"""The filtered score pass around its groups of rows (16 or 32), units (64 / 128 rows per wavefront, 256 / 512 per workgroup) and
chunks, which the pipelined loads run past at the end of every mid-region."""
import pytest

from paper_2604_05438_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["l3b_128k", "l1b_32k"])
@pytest.mark.parametrize("chunk,interleave", [(0, 0), (512, 1), (1024, 2), (2048, 1)])
def test_score_groups_at_every_end(shape, chunk, interleave):
    """Every score (exported), index set and output of a ragged batch, filtered pipeline forced; scores to 1e-5, the bar of
    parity_utils.  The longest problem fills several chunks; budgets from one token to a fifth of the mid-region."""
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

