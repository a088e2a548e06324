"""Host-side checks that need no GPU: the C-ABI library loads, exports every symbol that
include/tkphi.h declares, and its pure-host entry points validate arguments."""
import ctypes as C
import os
import re

import pytest

from paper_2604_05438_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "tkphi.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(tkphi_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = B.lib()
    names = _declared_symbols()
    assert set(names) == set(B.EXPORTS), names
    for n in names:
        assert getattr(lib, n) is not None


def test_budget_rules_match_paper_example():
    # K = max(0, ceil(r L) - |A|): 21 / 144 / 636 at 4k / 16k / 64k, 1 %, 20 anchors
    assert [B.tkphi_budget_paper(L, 100, 4, 16) for L in (4096, 16384, 65536)] == [21, 144, 636]
    assert B.tkphi_budget_paper(4096, 100, 4, 64) == 0
    assert B.tkphi_budget_mid(4096, 100, 4, 64) == 40
    assert [B.tkphi_budget_mid(131072, bp, 4, 64) for bp in (50, 100, 200, 400)] == [655, 1310, 2620, 5240]


def _cfg(**kw):
    base = dict(n_q_heads=32, n_kv_heads=8, d_head=64, d_phi=64, n_sink=4, n_tail=64, dtype="bf16",
                score_scale=0.125, phi_in_scale=0.35, phi_norm_coef=0.0625)
    base.update(kw)
    return B.make_config(**base)


def test_workspace_query_and_config_validation():
    assert B.tkphi_workspace_bytes(_cfg(), 1, 32768, 327) > 32 * 32700 * 4
    assert B.tkphi_workspace_bytes(_cfg(), 4, 32768, 327) > 4 * 32 * 32700 * 4
    for bad in (dict(d_head=96), dict(n_q_heads=30), dict(d_phi=20), dict(n_q_heads=128), dict(dtype=7),
                dict(n_sink=-1)):
        assert B.tkphi_workspace_bytes(_cfg(**bad), 1, 4096, 40) == 0
        assert B.tkphi_last_error() != ""
    assert B.tkphi_workspace_bytes(_cfg(), 1, 0, 0) == 0


def test_tuning_overrides_are_validated_and_change_the_geometry():
    base = B.tkphi_workspace_bytes(_cfg(), 1, 32768, 327)
    assert B.tkphi_workspace_bytes(_cfg(tuning={"build_chunk": 64}), 1, 32768, 327) > base   # more chunk partials
    for bad in ({"scan_chunk": -1}, {"scan_chunk": 1 << 20}, {"interleave": 3}, {"force_generic": 2}, {"mlp_mode": 5},
                {"build_chunk": -64}, {"select_mode": 3}, {"select_test": -1}):
        assert B.tkphi_workspace_bytes(_cfg(tuning=bad), 1, 32768, 327) == 0
        assert "tuning" in B.tkphi_last_error()
    cfg = _cfg()
    cfg.tuning.reserved[2] = 1
    assert B.tkphi_workspace_bytes(cfg, 1, 32768, 327) == 0


def test_mlp_feature_map_config_validation():
    mlp = dict(phi_kind=B.TKPHI_PHI_MLP, cache_features=1, d_emb=512)
    base = B.tkphi_workspace_bytes(_cfg(cache_features=1), 1, 32768, 327)
    with_mlp = B.tkphi_workspace_bytes(_cfg(**mlp), 1, 32768, 327)
    assert with_mlp > base > 0                     # activation block + packed weights of the MLP build
    # without a feature cache the build holds the features of a group of problems in the workspace
    assert B.tkphi_workspace_bytes(_cfg(**dict(mlp, cache_features=0)), 1, 32768, 327) > with_mlp
    assert B.tkphi_workspace_bytes(_cfg(**dict(mlp, cache_features=0, d_emb=64)), 1, 4096, 40) == 0   # (not a width that fuses)
    for bad in (dict(mlp, d_emb=96), dict(mlp, d_emb=32), dict(mlp, d_emb=2048), dict(mlp, dtype="f32"), dict(phi_kind=7)):
        assert B.tkphi_workspace_bytes(_cfg(**bad), 1, 4096, 40) == 0
        assert B.tkphi_last_error() != ""
    # the problem table must carry the MLP tables instead of Wq / Wk
    cfg = _cfg(**mlp)
    p = B.tkphi_problem(K=4096, V=8192, stride_head=1000 * 64, stride_tok=64, Wq=0, bq=0, Wk=0, bk=0, S=4096, u=4096,
                        q=4096, out=4096, topk_idx=0, aux=0, scores=0, phi_cache=4096, mlp_q=4096, mlp_k=4096,
                        L=1000, topk=9)
    B.tkphi_check_problems(cfg, (B.tkphi_problem * 1)(p), 1, 1000, 9, True)
    for field in ("mlp_q", "mlp_k", "phi_cache"):
        q = B.tkphi_problem.from_buffer_copy(p)
        setattr(q, field, 0)
        with pytest.raises(B.TkphiError):
            B.tkphi_check_problems(cfg, (B.tkphi_problem * 1)(q), 1, 1000, 9, True)
    # ... and no cache where the configuration has none
    q = B.tkphi_problem.from_buffer_copy(p)
    q.phi_cache = 0
    B.tkphi_check_problems(_cfg(**dict(mlp, cache_features=0)), (B.tkphi_problem * 1)(q), 1, 1000, 9, True)


def test_generated_token_bounds_are_validated():
    assert B.tkphi_workspace_bytes(_cfg(max_gen=64), 1, 4096, 40) >= B.tkphi_workspace_bytes(_cfg(), 1, 4096, 40) > 0
    assert B.tkphi_workspace_bytes(_cfg(max_gen=-1), 1, 4096, 40) == 0
    cfg = _cfg(max_gen=32)
    p = B.tkphi_problem(K=4096, V=8192, stride_head=1100 * 64, stride_tok=64, Wq=4096, bq=4096, Wk=4096, bk=4096,
                        S=4096, u=4096, q=4096, out=4096, L=1000, topk=9, n_gen=32)
    B.tkphi_check_problems(cfg, (B.tkphi_problem * 1)(p), 1, 1000, 9, True)
    for bad in (33, -1):
        q = B.tkphi_problem.from_buffer_copy(p)
        q.n_gen = bad
        with pytest.raises(B.TkphiError) as e:
            B.tkphi_check_problems(cfg, (B.tkphi_problem * 1)(q), 1, 1000, 9, True)
        assert e.value.status == B.TKPHI_ESHAPE


def test_status_strings():
    seen = {B.tkphi_status_string(s) for s in range(-6, 1)}
    assert len(seen) == 7 and B.tkphi_status_string(-99) == "unknown status"


def test_check_problems_rejects_bad_tables():
    cfg = _cfg()
    good = B.tkphi_problem(K=4096, V=8192, stride_head=1000 * 64, stride_tok=64, Wq=4096, bq=4096, Wk=4096,
                           bk=4096, S=4096, u=4096, q=4096, out=4096, topk_idx=0, aux=0, scores=0, L=1000, topk=9)
    arr = (B.tkphi_problem * 1)(good)
    B.tkphi_check_problems(cfg, arr, 1, 1000, 9, True)

    def expect(status, **kw):
        p = B.tkphi_problem.from_buffer_copy(good)
        for k, v in kw.items():
            setattr(p, k, v)
        with pytest.raises(B.TkphiError) as e:
            B.tkphi_check_problems(cfg, (B.tkphi_problem * 1)(p), 1, 1000, 9, True)
        assert e.value.status == status, e.value

    expect(B.TKPHI_EINVAL, K=0)
    expect(B.TKPHI_EINVAL, out=0)
    expect(B.TKPHI_EALIGN, V=8200)
    expect(B.TKPHI_EALIGN, stride_tok=65)
    expect(B.TKPHI_EALIGN, stride_tok=32)
    expect(B.TKPHI_ESHAPE, L=1001)
    expect(B.TKPHI_ESHAPE, L=0)
    expect(B.TKPHI_ESHAPE, topk=10)
    expect(B.TKPHI_ESHAPE, topk=-1)


def test_calls_reject_bad_arguments_before_any_launch():
    cfg = _cfg()
    lib = B.lib()
    nbytes = B.tkphi_workspace_bytes(cfg, 1, 1000, 9)
    # null workspace / too small / misaligned / bad mode / null table: all fail on the host
    assert lib.tkphi_decode(C.byref(cfg), 4096, 1, 1000, 9, 0, None, nbytes, None) == B.TKPHI_EWORKSPACE
    assert lib.tkphi_decode(C.byref(cfg), 4096, 1, 1000, 9, 0, 4096, nbytes - 1, None) == B.TKPHI_EWORKSPACE
    assert lib.tkphi_decode(C.byref(cfg), 4096, 1, 1000, 9, 0, 4100, nbytes, None) == B.TKPHI_EWORKSPACE
    assert lib.tkphi_decode(C.byref(cfg), 4096, 1, 1000, 9, 5, 4096, nbytes, None) == B.TKPHI_EINVAL
    assert lib.tkphi_decode(C.byref(cfg), None, 1, 1000, 9, 0, 4096, nbytes, None) == B.TKPHI_EINVAL
    assert lib.tkphi_build_summaries(C.byref(cfg), None, 1, 1000, 4096, nbytes, None) == B.TKPHI_EINVAL
    assert lib.tkphi_build_summaries(None, 4096, 1, 1000, 4096, nbytes, None) == B.TKPHI_EINVAL
    assert "null" in B.tkphi_last_error()
    # zero problems is a no-op
    assert lib.tkphi_decode(C.byref(cfg), None, 0, 1000, 9, 0, 4096, nbytes, None) == B.TKPHI_OK


@pytest.mark.parametrize("seed", range(6))
def test_reported_workspace_serves_every_mode_and_smaller_bounds(seed):
    """What tkphi_workspace_bytes reports for some bounds is accepted by decode calls in every mode, the diagnostics flag
    included, and, for one problem, by calls with a shorter sequence and no larger a share of it retrieved.  (The table pointer
    is misaligned, which is the last thing a call checks: EALIGN says that everything else passed, and nothing is enqueued.)
    Batches: also by half as many problems (several workgroups per head, and two sets of candidate lists, may come in there)."""
    import random
    r = random.Random(seed)
    lib = B.lib()
    for _ in range(400):
        d, hkv = r.choice([64, 128]), r.choice([1, 2, 4, 8])
        cfg = _cfg(n_q_heads=hkv * r.choice([1, 3, 4, 8]), n_kv_heads=hkv, d_head=d, d_phi=r.choice([d, d, d, 48]), dtype=r.choice(["bf16", "bf16", "f32"]),
                   cache_features=int(r.random() < 0.2))
        n = r.choice([1, 1, 2, 4, 6, 10, 16, 32, 64, 200])
        L = int(2 ** r.uniform(7, 17.3))
        K = int(L * 10 ** r.uniform(-3, -0.3))
        size = B.tkphi_workspace_bytes(cfg, n, L, K)
        assert size > 0
        calls = [(n, L, K, m | f) for m in (0, 1, 2) for f in (0, B.TKPHI_FLAG_DIAG)]
        if n > 1:
            calls.append((n // 2, L, K, 0))
        else:
            calls.append((1, L // 2, K // 2, 0))
        for m, l, k, mode in calls:
            st = lib.tkphi_decode(C.byref(cfg), 4100, m, l, k, mode, 4096, size, None)
            assert st == B.TKPHI_EALIGN, (n, L, K, m, l, k, mode, st, B.tkphi_last_error())


def test_reported_workspace_of_batches():
    """Batches with one workgroup per head lay their candidate lists out once (a rescan writes them over): against the spill
    pipeline's scores 8 bytes per head and token, not 16.  (Budgets of at most 1/64 report room for both sets.)"""
    w = dict(n_q_heads=32, n_kv_heads=8, d_head=64, d_phi=64)
    for n, L, K in ((256, 50000, 1000), (256, 131072, 5242), (40, 30000, 2100), (256, 4096, 327)):
        spill = B.tkphi_workspace_bytes(_cfg(tuning={"select_mode": 1}, **w), n, L, K)
        assert B.tkphi_workspace_bytes(_cfg(**w), n, L, K) <= 1.05 * (spill + n * 32 * L * 8)


@pytest.mark.parametrize("seed", range(4))
def test_reported_workspace_serves_shorter_builds(seed):
    """A summary build is accepted in the workspace that tkphi_workspace_bytes reports for any larger bounds.  Few query heads per KV head and
    small budgets: there the partials of the build decide the size, and their number goes up and down with the length and the number of
    problems.  (Misaligned table as above: EALIGN is acceptance.)"""
    import random
    r = random.Random(900 + seed)
    lib = B.lib()
    fixed = [(8, 64, 1, 11539, 1, 10126), (8, 64, 1, 15593, 1, 8212), (8, 64, 1, 21530, 1, 12261), (1, 64, 1, 101463, 1, 93995),
             (1, 128, 2, 12000, 2, 8000), (4, 64, 64, 4598, 51, 1503), (1, 128, 3, 199066, 2, 130670)]
    for i in range(1500):
        if i < len(fixed):
            hkv, d, n, L, n2, L2 = fixed[i]
            dtype, cache = "bf16", 0
        else:
            hkv, d, n = r.choice([1, 1, 2, 4, 8]), r.choice([64, 128]), r.choice([1, 1, 1, 2, 3, 4, 8, 16, 33, 64, 200])
            L = int(2 ** r.uniform(7, 18))
            n2, L2 = r.randint(1, n), r.randint(1, L)
            dtype, cache = r.choice(["bf16", "bf16", "f32"]), int(r.random() < 0.3)
        cfg = _cfg(n_q_heads=hkv * r.choice([1, 1, 2]), n_kv_heads=hkv, d_head=d, d_phi=d, dtype=dtype, cache_features=cache)
        size = B.tkphi_workspace_bytes(cfg, n, L, L // 100)
        for m, l in ((n2, L2), (n, L2), (n2, L), (n, L)):
            st = lib.tkphi_build_summaries(C.byref(cfg), 4100, m, l, 4096, size, None)
            assert st == B.TKPHI_EALIGN, (hkv, d, dtype, n, L, m, l, st, B.tkphi_last_error())
        # one chunk's partial of every KV head is too little for all but the shortest
        per = hkv * n * d * (d + 1) * 4
        if L > 8 * 4096 and n * hkv <= 8:
            assert lib.tkphi_build_summaries(C.byref(cfg), 4100, n, L, 4096, 4096 + per, None) == B.TKPHI_EWORKSPACE
