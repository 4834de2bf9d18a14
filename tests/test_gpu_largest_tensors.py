"""GPU, bf16: tensors next to 4 GiB, the largest that the attention takes (below 2^31 elements) -- on either side of the line from which rows are packed
because a row's byte offset and what the copies add to it no longer fit 32 bits."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import streaming_attention as O

from gpu_helpers import DEV, to_f64

pytestmark = pytest.mark.gpu

D = 128


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    yield st_
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n_tokens", [2 ** 24 - 17, 2 ** 24 - 1])
def test_tensors_next_to_four_gib(st, n_tokens):
    """One head of 128 dims: the first, a middle and the last sequence, of some hundred tokens, against the oracle."""
    long, short = W.tokens_from_segments([2000, 2096], [2048, 2048]), W.tokens_from_segments([70, 90], [80, 60])
    n_long, n_short = len(long[0]), len(short[0])
    count, rest = divmod(n_tokens - 3 * n_short, n_long)
    ragged = W.tokens_from_segments([rest // 2], [rest - rest // 2])
    order = [short] + [long] * (count // 2) + [short] + [long] * (count - count // 2) + [ragged, short]
    checked = (0, 1 + count // 2, len(order) - 1)
    cu = np.concatenate([[0], np.cumsum([len(s[0]) for s in order])]).astype(np.int32)
    assert cu[-1] == n_tokens
    streams, segments, positions = (torch.from_numpy(np.concatenate([s[i] for s in order]).astype(np.int32)).to(DEV) for i in range(3))
    gen = torch.Generator(device=DEV).manual_seed(95)
    q, k, v, g = (torch.empty((n_tokens, 1, D), dtype=torch.bfloat16, device=DEV).normal_(generator=gen) for _ in range(4))
    plan = st.st_plan_create(segments, streams, positions, cu).heads_per_workgroup(1)
    lse = torch.empty((n_tokens, 1), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(q, k, v, plan, lse=lse)
    grads = st.st_attn_prefill_bwd(g, q, k, v, out, lse, plan)
    ids = [x.astype(np.int32) for x in short]
    for b in checked:
        sl = slice(int(cu[b]), int(cu[b + 1]))
        x = [to_f64(t[sl]).astype(np.float32) for t in (q, k, v, g)]
        ref, _ = O.attention_dense(*x[:3], *ids)
        assert np.abs(to_f64(out[sl]) - ref).max() <= 2e-2, b                # (the parity suite's bound of bf16)
        refs = O.attention_varlen_backward(*x, *ids, np.array([0, n_short], np.int32))
        for name, got, want in zip(("dq", "dk", "dv"), grads, refs):
            # (the bound of the row-block tests: P, dS and the result are rounded to 4e-3 of their size)
            assert np.abs(to_f64(got[sl]) - want).max() <= 6e-2 * max(1.0, np.abs(want).max()), (b, name)
