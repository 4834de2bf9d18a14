"""GPU, fp32: Inf and NaN in the operands of a token reach the results of the pairs that the mask allows and no others -- a row's
output and gradients are bit for bit what they are without the bad value unless the row sees its token (forward, dQ) or is
seen through it (dK, dV)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import streaming_attention as O

from gpu_helpers import DEV, ids_to_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


# two sequences; streams of 51, 67, 70 and 33 tokens, so that the planted tokens sit inside, at the start and at the end of blocks
LISTS = [(np.array([20, 31]), np.array([25, 42])), (np.array([38, 32]), np.array([20, 13]))]
HEADS = [(4, 2, 64), (8, 2, 128), (2, 2, 128)]


def _case(hq, hkv, d):
    cfg = W._assemble("isolation", "f32", hq, hkv, d, LISTS, "interleaved", 41)
    seen = np.zeros((cfg.n_tokens, cfg.n_tokens), bool)           # [row, key]
    for b in range(cfg.batch):
        sl = slice(int(cfg.cu_seqlens[b]), int(cfg.cu_seqlens[b + 1]))
        seen[sl, sl] = O.dense_mask(cfg.stream_ids[sl], cfg.segment_ids[sl], cfg.positions[sl])
    # tokens to plant a value in: of the first sequence source tokens 0, 31, 40 and 50, reasoning tokens 0, 33 and 66; the second's last
    n0 = int(cfg.cu_seqlens[1])
    of = lambda stream: np.flatnonzero(cfg.stream_ids[:n0] == stream)
    tokens = [int(t) for t in (*of(0)[[0, 31, 40, 50]], *of(1)[[0, 33, 66]], cfg.n_tokens - 1)]
    x = {n: to_dev(t, "f32") for n, t in zip("qkv", cfg.tensors())}
    x["g"] = to_dev(W.normal(np.random.Generator(np.random.PCG64(42)), tuple(x["q"].shape), "f32"), "f32")
    return cfg, torch.from_numpy(seen).to(DEV), tokens, x


def _planted(x, name, token, value, whole):
    """The operands with `value` in one element, or in all, of the token's row of one of them."""
    y = dict(x)
    y[name] = x[name].clone()
    if whole:
        y[name][token] = value
    else:
        y[name][token, 0, 5] = value
    return y


@pytest.mark.parametrize("value,whole", [(float("inf"), False), (float("nan"), True)])
@pytest.mark.parametrize("hq,hkv,d", HEADS)
def test_forward_rows_that_do_not_see_the_token(st, hq, hkv, d, value, whole):
    cfg, seen, tokens, x = _case(hq, hkv, d)
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)

    def forward(y):
        lse = torch.empty((cfg.n_tokens, hq), dtype=torch.float32, device=DEV)
        return st.st_attn_prefill(y["q"], y["k"], y["v"], plan, lse=lse), lse

    out, lse = forward(x)
    for name in "kv":
        for t in tokens:
            bad_out, bad_lse = forward(_planted(x, name, t, value, whole))
            others = ~seen[:, t]
            assert torch.equal(bad_out[others], out[others]) and torch.equal(bad_lse[others], lse[others]), (name, t)
            if name == "v":                # ... and every row that sees it shows it, in the planted dim
                assert not torch.isfinite(bad_out[~others, 0, 5]).any(), t


@pytest.mark.parametrize("value,whole", [(float("inf"), False), (float("nan"), True)])
@pytest.mark.parametrize("hq,hkv,d", HEADS)
def test_gradients_of_pairs_without_the_token(st, hq, hkv, d, value, whole):
    cfg, seen, tokens, x = _case(hq, hkv, d)
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    lse = torch.empty((cfg.n_tokens, hq), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(x["q"], x["k"], x["v"], plan, lse=lse)
    backward = lambda y: st.st_attn_prefill_bwd(y["g"], y["q"], y["k"], y["v"], out, lse, plan)       # (out and lse: the finite ones)
    finite = backward(x)
    everything = torch.ones(cfg.n_tokens, dtype=torch.bool, device=DEV)
    for name in "qkvg":
        for t in tokens:
            itself = torch.zeros_like(everything)
            itself[t] = True
            # a key's value enters dQ of the rows that see it and its own dK (dV too if it is the key itself); a row's, its own dQ
            # and dK, dV of the keys that it sees
            untouched = ((~seen[:, t], ~itself, ~itself if name == "k" else everything) if name in "kv" else
                         (~itself, ~seen[t], ~seen[t]))
            for which, got, want, rows in zip(("dq", "dk", "dv"), backward(_planted(x, name, t, value, whole)), finite, untouched):
                assert torch.equal(got[rows], want[rows]), (name, t, which)
            if whole and name == "v":
                assert torch.isnan(backward(_planted(x, name, t, value, whole))[0][seen[:, t]]).all()
