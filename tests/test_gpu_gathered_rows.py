"""GPU, bf16: the prefill's one-head form and the gradients take their rows straight from the tensors, token by token.  Streams that end around a
tile's 64 rows, numbers of KV heads that are no power of two, and neighbours that must not be touched: the sequences before and
after hold NaN alone, and a row past a stream's end would bring one in."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import streaming_attention as O

from gpu_helpers import DEV, ids_to_dev, to_dev, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("hq,hkv,d", [(3, 3, 128), (10, 5, 64), (4, 1, 128), (2, 2, 64)])
@pytest.mark.parametrize("src,rsn", [(1, 1), (63, 65), (64, 128), (65, 63), (129, 0), (0, 191), (200, 257)])
def test_rows_of_their_own_stream_alone(st, hq, hkv, d, src, rsn, fused):
    lists = [(np.array([70]), np.array([60])), (np.array([src // 2, src - src // 2]), np.array([rsn // 3, rsn - rsn // 3])), (np.array([5]), np.array([9]))]
    cfg = W._assemble("gathered", "bf16", hq, hkv, d, lists, "interleaved", 71)
    q, k, v = cfg.tensors()
    own = slice(int(cfg.cu_seqlens[1]), int(cfg.cu_seqlens[2]))
    others = np.r_[0:own.start, own.stop:cfg.n_tokens]
    tq, tk, tv = (to_dev(x, "bf16") for x in (q, k, v))
    for t in (tk, tv):
        t[torch.from_numpy(others).to(DEV)] = float("nan")
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens).heads_per_workgroup(1)
    lse = torch.empty((cfg.n_tokens, hq), dtype=torch.float32, device=DEV)
    if fused:
        out = st.st_attn_prefill_rope(tq, tk, tv, torch.from_numpy(cfg.positions).to(DEV), cfg.theta, plan, lse=lse)
        q, k = O.rope(q, cfg.positions, cfg.theta), O.rope(k, cfg.positions, cfg.theta)
    else:
        out = st.st_attn_prefill(tq, tk, tv, plan, lse=lse)
    ref, ref_lse = O.attention_dense(q[own], k[own], v[own], cfg.stream_ids[own], cfg.segment_ids[own], cfg.positions[own])
    # the parity suite's bound of bf16 (rotated keys and queries are rounded once more)
    tol = 4e-2 if fused else 2e-2
    assert np.abs(to_f64(out[own]) - ref).max() <= tol
    assert np.abs(to_f64(lse[own]) - ref_lse).max() <= tol


@pytest.mark.parametrize("hq,hkv,d", [(3, 3, 128), (10, 5, 64), (4, 1, 128), (8, 2, 64)])
@pytest.mark.parametrize("src,rsn", [(1, 1), (63, 65), (64, 128), (65, 63), (129, 0), (0, 191), (200, 257)])
def test_gradients_of_their_own_stream_alone(st, hq, hkv, d, src, rsn):
    lists = [(np.array([70]), np.array([60])), (np.array([src // 2, src - src // 2]), np.array([rsn // 3, rsn - rsn // 3])), (np.array([5]), np.array([9]))]
    cfg = W._assemble("gathered", "bf16", hq, hkv, d, lists, "interleaved", 72)
    q, k, v = cfg.tensors()
    g = W.normal(np.random.Generator(np.random.PCG64(73)), q.shape, "bf16")
    own = slice(int(cfg.cu_seqlens[1]), int(cfg.cu_seqlens[2]))
    others = torch.from_numpy(np.r_[0:own.start, own.stop:cfg.n_tokens]).to(DEV)
    tq, tk, tv, tg = (to_dev(x, "bf16") for x in (q, k, v, g))
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    lse = torch.empty((cfg.n_tokens, hq), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(tq, tk, tv, plan, lse=lse)
    for t in (tq, tk, tv, tg, out, lse):
        t[others] = float("nan")
    grads = st.st_attn_prefill_bwd(tg, tq, tk, tv, out, lse, plan)
    refs = O.attention_varlen_backward(q, k, v, g, cfg.stream_ids, cfg.segment_ids, cfg.positions, cfg.cu_seqlens)
    for name, got, ref in zip(("dq", "dk", "dv"), grads, refs):
        # (the bound of the row-block tests: P, dS and the result are rounded to 4e-3 of their size)
        assert np.abs(to_f64(got[own]) - ref[own]).max() <= 6e-2 * max(1.0, np.abs(ref[own]).max()), name


@pytest.mark.parametrize("fused,hq,hkv,d,tokens", [(True, 4, 2, 128, 3600), (True, 3, 3, 64, 3600), (False, 8, 1, 128, 5100), (True, 4, 2, 128, 3400)])
def test_long_sequences_on_either_side_of_the_packed_tiles(st, fused, hq, hkv, d, tokens):
    """One head per wave over packed tiles and over gathered rows: sampled rows against the oracle."""
    cfg = W._assemble("long", "bf16", hq, hkv, d, [(np.array([tokens // 4, tokens // 8]), np.array([tokens // 3, tokens - tokens // 4 - tokens // 8 - tokens // 3]))], "interleaved", 74)
    q, k, v = cfg.tensors()
    tq, tk, tv = (to_dev(x, "bf16") for x in (q, k, v))
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens).heads_per_workgroup(1)
    if fused:
        out = st.st_attn_prefill_rope(tq, tk, tv, torch.from_numpy(cfg.positions).to(DEV), cfg.theta, plan)
        q, k = O.rope(q, cfg.positions, cfg.theta), O.rope(k, cfg.positions, cfg.theta)
    else:
        out = st.st_attn_prefill(tq, tk, tv, plan)
    got = to_f64(out)
    mask = O.dense_mask(cfg.stream_ids, cfg.segment_ids, cfg.positions)
    for row in (0, 1, 63, tokens // 4, tokens // 2, tokens - 65, tokens - 1):
        for h in range(hq):
            s = np.where(mask[row], k[:, h // (hq // hkv)].astype(np.float64) @ q[row, h].astype(np.float64) / np.sqrt(d), -np.inf)
            p = np.exp(s - s.max())
            ref = (p / p.sum()) @ v[:, h // (hq // hkv)].astype(np.float64)
            assert np.abs(got[row, h] - ref).max() <= (4e-2 if fused else 2e-2), (row, h)


@pytest.mark.parametrize("hq,hkv,d", [(5, 5, 128), (12, 6, 64), (8, 8, 128), (7, 7, 64), (1, 1, 128)])
def test_rotated_keys_of_several_heads_per_workgroup(st, hq, hkv, d):
    """From 4,096 (key tile, head) pairs on a workgroup rotates four heads, the last one what is left of them: the batch as a whole
    against its parts, which have fewer, bit for bit, and three sequences against the oracle."""
    rng = np.random.Generator(np.random.PCG64(75))
    per_part, pairs = -(-4096 // (4 * 2 * hkv)), 0
    lists = [(rng.integers(0, 60, 2), rng.integers(1, 60, 2)) for _ in range(4 * per_part)]
    for s, r in lists:
        pairs += (-(-int(s.sum() + r.sum()) // 64) + 1) * hkv
    cfg = W._assemble("short", "bf16", hq, hkv, d, lists, "interleaved", 76)
    q, k, v = cfg.tensors()
    tq, tk, tv = (to_dev(x, "bf16") for x in (q, k, v))
    ids = (*ids_to_dev(cfg),)

    def run(b0, b1):
        sl = slice(int(cfg.cu_seqlens[b0]), int(cfg.cu_seqlens[b1]))
        plan = st.st_plan_create(*(x[sl].contiguous() for x in ids), cfg.cu_seqlens[b0:b1 + 1] - cfg.cu_seqlens[b0]).heads_per_workgroup(1)
        return st.st_attn_prefill_rope(tq[sl], tk[sl], tv[sl], ids[2][sl].contiguous(), cfg.theta, plan)

    assert pairs >= 4096 > pairs / 4 * 1.2
    whole = run(0, len(lists))
    parts = [run(p * per_part, (p + 1) * per_part) for p in range(4)]
    assert torch.equal(whole, torch.cat(parts))
    for b in (0, len(lists) // 2, len(lists) - 1):
        sl = slice(int(cfg.cu_seqlens[b]), int(cfg.cu_seqlens[b + 1]))
        ref, _ = O.attention_dense(O.rope(q[sl], cfg.positions[sl], cfg.theta), O.rope(k[sl], cfg.positions[sl], cfg.theta), v[sl], cfg.stream_ids[sl],
                                   cfg.segment_ids[sl], cfg.positions[sl])
        assert np.abs(to_f64(whole[sl]) - ref).max() <= 4e-2, b
