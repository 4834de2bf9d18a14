"""GPU: attention and its gradients at the edges of the kernels' row blocks -- streams one token short of, exactly and one
token past a multiple of the 32 rows a wave owns, single tokens, and rows whose visible source prefix ends inside a block --
against the fp64 oracle."""
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


# per sequence: (source segment lengths, reasoning segment lengths)
EDGES = [(np.array([1]), np.array([1])), (np.array([31, 1]), np.array([32, 1])), (np.array([33]), np.array([63])),
         (np.array([30, 35]), np.array([1, 96])), (np.array([127, 1, 1]), np.array([31, 97, 1])), (np.array([0]), np.array([161]))]


def _case(dtype, hq, hkv, d, layout):
    return W._assemble("edges", dtype, hq, hkv, d, EDGES, layout, 21)


def _forward_and_backward(st, cfg, heads=0):
    q, k, v = cfg.tensors()
    g = W.normal(np.random.Generator(np.random.PCG64(22)), q.shape, cfg.dtype)
    tq, tk, tv, tg = (to_dev(x, cfg.dtype) for x in (q, k, v, g))
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens).heads_per_workgroup(heads)
    lse = torch.empty((cfg.n_tokens, cfg.n_q_heads), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(tq, tk, tv, plan, lse=lse)
    grads = st.st_attn_prefill_bwd(tg, tq, tk, tv, out, lse, plan)
    torch.cuda.synchronize()
    refs = O.attention_varlen_backward(q, k, v, g, cfg.stream_ids, cfg.segment_ids, cfg.positions, cfg.cu_seqlens)
    return (q, k, v), out, lse, grads, refs


def _check(cfg, inputs, out, lse, grads, refs):
    # forward: the bounds of the parity suite (1e-4 for fp32 inputs, 2e-2 for bf16).  Gradients: an entry sums at most
    # 161 x 8 terms; fp32 rounds each to 6e-8 of its size (2e-4 is far above), bf16 rounds P, dS and the result to 4e-3.
    q, k, v = inputs
    tol, tol_g = (1e-4, 2e-4) if cfg.dtype == "f32" else (2e-2, 6e-2)
    for b in range(cfg.batch):
        sl = slice(int(cfg.cu_seqlens[b]), int(cfg.cu_seqlens[b + 1]))
        ref, ref_lse = O.attention_dense(q[sl], k[sl], v[sl], cfg.stream_ids[sl], cfg.segment_ids[sl], cfg.positions[sl])
        assert np.abs(to_f64(out[sl]) - ref).max() <= tol, b
        assert np.abs(to_f64(lse[sl]) - ref_lse).max() <= tol, b
    for name, got, ref in zip(("dq", "dk", "dv"), grads, refs):
        assert np.abs(to_f64(got) - ref).max() <= tol_g * max(1.0, np.abs(ref).max()), name


@pytest.mark.parametrize("hq,hkv,d,layout", [(2, 1, 64, "interleaved"), (4, 4, 128, "grouped"), (8, 2, 128, "interleaved"), (8, 1, 64, "grouped")])
def test_fp32_row_blocks(st, hq, hkv, d, layout):
    """(The key side of the backward splits the query heads of a group two, one, four and eight ways here.)"""
    cfg = _case("f32", hq, hkv, d, layout)
    _check(cfg, *_forward_and_backward(st, cfg))


@pytest.mark.parametrize("hq,hkv,d", [(16, 2, 64), (4, 2, 128), (6, 1, 128), (3, 3, 64)])
def test_key_side_split_over_query_heads(st, hq, hkv, d):
    """Few KV heads under sequences of 512 tokens and more: the key side of the backward splits the query heads of a group
    over several workgroups (8, 2 and 6 ways here, and not at all with one head per group) and adds their sums."""
    lists = [(np.array([127, 130]), np.array([129, 200])), (np.array([300]), np.array([260]))]
    cfg = W._assemble("split", "bf16", hq, hkv, d, lists, "interleaved", 23)
    _check(cfg, *_forward_and_backward(st, cfg))


@pytest.mark.parametrize("heads", [1, 2])
@pytest.mark.parametrize("hq,hkv,d", [(3, 3, 128), (4, 2, 64), (8, 2, 128), (16, 2, 64), (12, 2, 128)])
def test_query_heads_over_waves(st, hq, hkv, d, heads):
    """The waves of a workgroup take one, two or four sets of one or two query heads of a KV head and 128, 64 or 32 rows of
    an item (groups of 1, 2, 4, 8 and 6 heads), rows and visible prefixes ending inside the parts."""
    cfg = _case("bf16", hq, hkv, d, "interleaved")
    _check(cfg, *_forward_and_backward(st, cfg, heads))


@pytest.mark.parametrize("lens,hq,hkv,d,parts", [([760] * 8, 16, 8, 128, 1), ([2400] * 3, 16, 8, 128, 1), ([914] * 10, 16, 8, 64, 1), ([2700] * 2, 16, 8, 128, 2),
                                                 ([6100], 16, 2, 128, 8), ([1700] * 10, 16, 2, 64, 4), ([150] * 8, 8, 1, 128, 1), ([760] * 8, 40, 8, 128, 1),
                                                 # ragged batches: the longest sequence holds the launch up
                                                 ([6000] + [300] * 8, 8, 4, 128, 2), ([6000] + [300] * 8, 16, 2, 64, 8), ([3000] + [600] * 10, 16, 8, 64, 2),
                                                 ([333, 2005, 2327, 387, 925, 1831, 1080, 2878, 503, 1074], 16, 2, 64, 8)])
def test_parts_of_the_key_side(st, lens, hq, hkv, d, parts):
    """How many ways the key side splits the query heads of a group, as the workspace tells: each part has fp32 sums of its own,
    behind delta, the row statistics and the row tiles of all heads."""
    cfg = W._assemble("parts", "bf16", hq, hkv, d, [(np.array([n // 2]), np.array([n - n // 2])) for n in lens], "grouped", 24)
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    up = lambda n: (n + 255) // 256 * 256
    tiles = sum((n + 63) // 64 + 1 for n in lens)
    base = up(cfg.n_tokens * hq * 4) + up(tiles * hq * 1024) + 2 * (up(tiles * hkv * 64 * d * 2) + up(tiles * hq * 64 * d * 2)) + 256
    sums = up(2 * parts * cfg.n_tokens * hkv * d * 4) if parts > 1 else 0
    assert int(st.load_library().st_prefill_bwd_workspace_bytes(plan.handle, hq, hkv, d, st.ST_BF16)) == base + sums


@pytest.mark.parametrize("dtype,hq,hkv,d", [("bf16", 8, 2, 128), ("bf16", 4, 2, 64), ("bf16", 3, 3, 128), ("f32", 4, 2, 128), ("f32", 2, 1, 64)])
@pytest.mark.parametrize("longest", [1, 32, 33, 64, 65, 96, 97])
def test_no_sequence_fills_an_item(st, dtype, hq, hkv, d, longest):
    """Launches without workgroups for the parts of an item that no sequence has rows for: all of the longest sequence in one stream,
    in the other, or in both; sequences of one token beside it."""
    split = lambda s, r: (np.array([s], dtype=np.int64), np.array([r], dtype=np.int64))
    lists = [split(longest, 0), split(0, longest), split(longest // 2, longest - longest // 2), split(1, 0), split(0, 1)]
    cfg = W._assemble("short", dtype, hq, hkv, d, lists, "grouped", 25 + longest)
    _check(cfg, *_forward_and_backward(st, cfg))
