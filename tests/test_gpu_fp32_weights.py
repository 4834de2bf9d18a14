"""GPU, fp32: single weights exp(score - reference) of the forward and of both gradient kernels, out of inputs that leave nothing else to round --
scores are one product with 1, values and incoming gradients pick one weight per dim."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import streaming_attention as O

from gpu_helpers import DEV, ids_to_dev, to_dev, to_f64

pytestmark = pytest.mark.gpu

N, BATCH = 31, 12              # tokens of a sequence: one block of 32, so that one wave holds every weight of a row


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


@pytest.mark.parametrize("hq,hkv,d", [(1, 1, 64), (1, 1, 128), (2, 1, 128)])
@pytest.mark.parametrize("lo,hi", [(-4, -1), (-12, -5), (-16, -11)])
def test_single_weights(st, hq, hkv, d, lo, hi):
    """A weight's error: 0.85e-7 of the exponential, 0.2e-7 of its bf16 terms and 0.6e-7 of their sum; the forward scales by 1 / sum, which rounds the
    weight and the one it is compared with, the row's first (1), by 0.6e-7 each."""
    cfg = W._assemble("weights", "f32", hq, hkv, d, [(np.array([N]), np.array([0]))] * BATCH, "interleaved", 81)
    x = np.random.Generator(np.random.PCG64(82)).uniform(lo, hi, (BATCH, N)).astype(np.float32)
    x[:, 0] = 0.0                                                  # the row's largest score
    k = np.zeros((BATCH, N, hkv, d), np.float32)
    q = np.zeros((BATCH, N, hq, d), np.float32)
    v = np.zeros((BATCH, N, hkv, d), np.float32)
    g = np.zeros((BATCH, N, hq, d), np.float32)
    at = np.arange(N)
    k[:, :, :, 0] = x[:, :, None]
    q[:, :, :, 0] = 1.0
    k[:, at[1:], :, at[1:]] = 1.0                                  # dims that the queries do not have pick a key's weight in dq
    q[:, at, :, 32 + at] = 1.0                                     # ... and these, which the keys do not have, a row's in dk
    v[:, at, :, at] = 1.0
    g[:, at, :, at] = 1.0
    flat = lambda t: to_dev(t.reshape(BATCH * N, -1, d), "f32")
    tq, tk, tv, tg = (flat(t) for t in (q, k, v, g))
    ones = flat(np.broadcast_to(v.max(axis=1, keepdims=True).max(axis=2, keepdims=True), q.shape))      # every key's dP is 1
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    out = to_f64(st.st_attn_prefill(tq, tk, tv, plan, scale=1.0)).reshape(BATCH, N, hq, d)
    zero_out, zero_lse = torch.zeros_like(tq), torch.zeros((BATCH * N, hq), dtype=torch.float32, device=DEV)
    dv = st.st_attn_prefill_bwd(tg, tq, tk, tv, zero_out, zero_lse, plan, scale=1.0)[2]
    dq, dk, _ = st.st_attn_prefill_bwd(ones, tq, tk, tv, zero_out, zero_lse, plan, scale=1.0)
    dq, dk, dv = (to_f64(t).reshape(BATCH, N, -1, d) for t in (dq, dk, dv))
    mask = O.dense_mask(cfg.stream_ids[:N], cfg.segment_ids[:N], cfg.positions[:N])
    i, j = np.nonzero(mask)
    i, j = i[j > 0], j[j > 0]
    want = np.exp(x.astype(np.float64))[:, j]                      # [sequence, pair]
    for h in range(hq):
        got = out[:, i, h, j] / out[:, i, h, 0]
        assert (np.abs(got - want) <= 2.9e-7 * want).all(), ("forward", h, np.abs(got / want - 1).max())
        got = dq[:, i, h, j]
        assert (np.abs(got - want) <= 1.7e-7 * want).all(), ("dq", h, np.abs(got / want - 1).max())
    for name, got in (("dk", dk[:, j, 0, 32 + i]), ("dv", dv[:, j, 0, i])):                   # (sums over the query heads, all alike)
        assert (np.abs(got - hq * want) <= 1.7e-7 * hq * want).all(), (name, np.abs(got / (hq * want) - 1).max())
