"""GPU, fp32: the kernels multiply operands that are split into three bf16 terms.  Values of any size keep fp32's precision, down to the
smallest, and finite values that the terms cannot hold, or whose products overflow as terms, are multiplied as fp32 has them."""
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


def _grads_64(cfg, q, k, v, g):
    """Output and gradients in 64 bits, and for every entry the sum of the sizes that it is made of: rounding errors are a part of that."""
    hq, group, d = q.shape[1], q.shape[1] // k.shape[1], q.shape[2]
    names = ("out", "dq", "dk", "dv")
    ref = {n: np.zeros(x.shape) for n, x in zip(names, (q, q, k, v))}
    room = {n: np.zeros(x.shape) for n, x in zip(names, (q, q, k, v))}
    scale = 1 / np.sqrt(d)
    for b in range(cfg.batch):
        sl = slice(int(cfg.cu_seqlens[b]), int(cfg.cu_seqlens[b + 1]))
        mask = O.dense_mask(cfg.stream_ids[sl], cfg.segment_ids[sl], cfg.positions[sl])
        for h in range(hq):
            hk = h // group
            q1, k1, v1, g1 = (x.astype(np.float64) for x in (q[sl, h], k[sl, hk], v[sl, hk], g[sl, h]))
            s = np.where(mask, q1 @ k1.T * scale, -np.inf)
            p = np.exp(s - s.max(1, keepdims=True))
            p /= p.sum(1, keepdims=True)
            out = p @ v1
            ds = p * (g1 @ v1.T - (g1 * out).sum(1, keepdims=True)) * scale
            ds_room = p * (np.abs(g1) @ np.abs(v1).T + (np.abs(g1) * np.abs(out)).sum(1, keepdims=True)) * scale
            ref["out"][sl, h], room["out"][sl, h] = out, p @ np.abs(v1)
            ref["dq"][sl, h], room["dq"][sl, h] = ds @ k1, ds_room @ np.abs(k1)
            ref["dk"][sl, hk] += ds.T @ q1
            room["dk"][sl, hk] += ds_room.T @ np.abs(q1)
            ref["dv"][sl, hk] += p.T @ g1
            room["dv"][sl, hk] += p.T @ np.abs(g1)
    return ref, room


def _check(st, cfg, q, k, v, g):
    """Entry by entry within 1e-5 of the sizes that it is made of (scores of up to 6 with an error of 5e-7 each enter every weight)."""
    tq, tk, tv, tg = (to_dev(x, "f32") for x in (q, k, v, g))
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    lse = torch.empty((cfg.n_tokens, q.shape[1]), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(tq, tk, tv, plan, lse=lse)
    got = dict(zip(("out", "dq", "dk", "dv"), (out, *st.st_attn_prefill_bwd(tg, tq, tk, tv, out, lse, plan))))
    ref, room = _grads_64(cfg, q, k, v, g)
    for name in got:
        x = to_f64(got[name])
        assert np.isfinite(x).all(), name
        # (2^-149: a result may be subnormal)
        assert (np.abs(x - ref[name]) <= 1e-5 * room[name] + 2.0 ** -149).all(), (name, (np.abs(x - ref[name]) / room[name]).max())


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 64), (3, 1, 128), (4, 2, 128)])
@pytest.mark.parametrize("where", ["odd dims of all", "values", "incoming gradients"])
def test_numbers_next_to_the_smallest(st, hq, hkv, d, where):
    """Operands of 2^-118: their last bits lie below the numbers that bf16 has, their products with one another and the results do not."""
    cfg = _case(hq, hkv, d)
    q, k, v = cfg.tensors()
    g = W.normal(np.random.Generator(np.random.PCG64(63)), q.shape, "f32")
    size = np.float32(2.0 ** -118)
    if where == "values":
        v = v * size
    elif where == "incoming gradients":
        g = g * size
    else:
        for x in (q, k, v, g):
            x[..., 1::2] *= size
    _check(st, cfg, q, k, v, g)


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 64), (4, 2, 64), (3, 1, 128), (4, 2, 128)])       # (one head per KV head: dK, dV in one part, else in parts)
@pytest.mark.parametrize("name,value", [("q", 3e31), ("k", -3e31), ("v", 3e31), ("v", -3.4e38), ("g", 3.4e38), ("g", -3e31)])
@pytest.mark.parametrize("token", [0, 40, 117])
def test_numbers_beyond_the_terms(st, hq, hkv, d, name, value, token):
    """A finite value that three bf16 terms cannot hold (from 2^104 = 2.03e31 on), in one element of a token; the dim it meets holds values
    of 2^-104, so that scores and gradients are finite and ordinary."""
    cfg = _case(hq, hkv, d)
    q, k, v = cfg.tensors()
    x = {"q": q, "k": k, "v": v, "g": W.normal(np.random.Generator(np.random.PCG64(64)), q.shape, "f32")}
    x[name][token, 0, 5] = value
    x[{"q": "k", "k": "q", "v": "g", "g": "v"}[name]][:, :, 5] *= np.float32(2.0 ** -104)
    _check(st, cfg, x["q"], x["k"], x["v"], x["g"])


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 64), (4, 2, 128)])
@pytest.mark.parametrize("token", [0, 40, 117])
def test_value_beyond_bf16(st, hq, hkv, d, token):
    """bf16 rounds up to Inf from (2 - 2^-8) 2^127 = 3.3962e38 on."""
    cfg = _case(hq, hkv, d)
    q, k, v = cfg.tensors()
    big = v.copy()
    big[token, 0, 5] = 3.4e38
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
