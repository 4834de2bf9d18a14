"""GPU, fp32: the kernels multiply operands that are split into three bf16 terms.  Values of any size keep fp32's precision, and a
finite value that bf16 has no number for (above 3.3895e38) is multiplied as fp32 has it."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import streaming_attention as O

from gpu_helpers import DEV, ids_to_dev, to_dev, to_f64

pytestmark = pytest.mark.gpu

LISTS = [(np.array([20, 31]), np.array([25, 42])), (np.array([1, 64]), np.array([33, 2]))]


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


def _case(hq, hkv, d):
    return W._assemble("split", "f32", hq, hkv, d, LISTS, "interleaved", 61)


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 64), (3, 1, 128), (4, 2, 128)])
def test_dims_of_unlike_size(st, hq, hkv, d):
    """Values and incoming gradients whose dims lie between 2^-48 and 2^48: every result entry is a sum of products of its own dim (out,
    dV), so its error is bounded by the sum of their sizes times the error of the weights -- 1e-5: scores of up to 6 with an error
    of 5e-7 each -- whatever the other dims hold."""
    cfg = _case(hq, hkv, d)
    q, k, v = cfg.tensors()
    size = (2.0 ** np.round(np.linspace(-48, 48, d))).astype(np.float32)
    g = W.normal(np.random.Generator(np.random.PCG64(62)), q.shape, "f32")
    v, g = v * size, g / size
    tq, tk, tv, tg = (to_dev(x, "f32") for x in (q, k, v, g))
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    lse = torch.empty((cfg.n_tokens, hq), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(tq, tk, tv, plan, lse=lse)
    dv = st.st_attn_prefill_bwd(tg, tq, tk, tv, out, lse, plan)[2]
    group = hq // hkv
    for b in range(cfg.batch):
        sl = slice(int(cfg.cu_seqlens[b]), int(cfg.cu_seqlens[b + 1]))
        mask = O.dense_mask(cfg.stream_ids[sl], cfg.segment_ids[sl], cfg.positions[sl])
        for h in range(hq):
            s = np.where(mask, q[sl, h].astype(np.float64) @ k[sl, h // group].astype(np.float64).T / np.sqrt(d), -np.inf)
            p = np.exp(s - s.max(1, keepdims=True))
            p /= p.sum(1, keepdims=True)
            v64 = v[sl, h // group].astype(np.float64)
            assert (np.abs(to_f64(out[sl, h]) - p @ v64) <= 1e-5 * (p @ np.abs(v64))).all(), (b, h)
        for hk in range(hkv):
            want, room = 0.0, 0.0
            for h in range(hk * group, (hk + 1) * group):
                s = np.where(mask, q[sl, h].astype(np.float64) @ k[sl, hk].astype(np.float64).T / np.sqrt(d), -np.inf)
                p = np.exp(s - s.max(1, keepdims=True))
                p /= p.sum(1, keepdims=True)
                want, room = want + p.T @ g[sl, h].astype(np.float64), room + p.T @ np.abs(g[sl, h].astype(np.float64))
            assert (np.abs(to_f64(dv[sl, hk]) - want) <= 1e-5 * room).all(), (b, hk)


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 64), (4, 2, 128)])
@pytest.mark.parametrize("token", [0, 40, 117])
def test_value_beyond_bf16(st, hq, hkv, d, token):
    cfg = _case(hq, hkv, d)
    q, k, v = cfg.tensors()
    big = v.copy()
    big[token, 0, 5] = 3.395e38
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    tq, tk = to_dev(q, "f32"), to_dev(k, "f32")
    out, out_big = (st.st_attn_prefill(tq, tk, to_dev(x, "f32"), plan) for x in (v, big))
    b = 0 if token < int(cfg.cu_seqlens[1]) else 1
    sl = slice(int(cfg.cu_seqlens[b]), int(cfg.cu_seqlens[b + 1]))
    seen = torch.zeros(cfg.n_tokens, dtype=torch.bool, device=DEV)
    seen[sl] = torch.from_numpy(O.dense_mask(cfg.stream_ids[sl], cfg.segment_ids[sl], cfg.positions[sl])[:, token - sl.start]).to(DEV)
    assert torch.equal(out_big[~seen], out[~seen])
    ref, _ = O.attention_dense(q[sl], k[sl], big[sl], cfg.stream_ids[sl], cfg.segment_ids[sl], cfg.positions[sl])
    got = to_f64(out_big[sl])
    assert np.isfinite(got).all()
    # (the planted dim's error is the weight's, relative to a result that the planted value makes up; the other dims: the parity bound)
    planted = np.abs(ref) > 1e30
    assert (np.abs(got - ref)[planted] <= 1e-5 * np.abs(ref)[planted]).all()
    assert np.abs(got - ref)[~planted].max() <= 1e-4
