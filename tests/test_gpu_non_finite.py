"""GPU: non-finite values go where the mask lets them and nowhere else -- a NaN key that a decode step sees makes its rows NaN,
however its token is dealt out over waves and units."""
import numpy as np
import pytest
import torch

import workloads as W

from gpu_helpers import DEV, make_cache, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


# a source cache whose last token is alone in its step of 32 tokens (64 for 8-bit caches), which is a wave's only one, or alone in
# the cache; reasoning caches that make the step one launch (both caches short) or two
@pytest.mark.parametrize("q_len,hq,hkv,d,fp8,n_src,n_rsn", [(1, 4, 2, 128, False, 33, 100), (1, 4, 2, 64, False, 33, 1500), (4, 8, 2, 128, False, 33, 1500),
                                                            (8, 8, 2, 128, False, 33, 1500), (8, 8, 2, 64, False, 33, 100), (1, 4, 2, 128, True, 65, 1500),
                                                            (1, 4, 2, 128, False, 1, 1500), (8, 8, 2, 64, False, 1, 1500)])
def test_visible_nan_key_reaches_its_rows(st, q_len, hq, hkv, d, fp8, n_src, n_rsn):
    rng = np.random.Generator(np.random.PCG64(480))
    caches = st.DualCache(*(make_cache(2, (n + 15) // 16, hkv, d, rng, fp8=fp8)[0] for n in (n_src, n_rsn)))
    lens = {}
    for which, n in ((st.ST_SOURCE, n_src), (st.ST_REASONING, n_rsn)):
        lens[which] = torch.tensor([n, n], dtype=torch.int32, device=DEV)
        st.st_kv_append(caches, which, *(to_dev(W.normal(rng, (2, n, hkv, d), "bf16"), "bf16") for _ in range(2)), lens[which])
    q = to_dev(W.normal(rng, (2, q_len, hq, d), "bf16"), "bf16")
    step = lambda: st.st_attn_decode_dual(q, caches, lens[st.ST_SOURCE], lens[st.ST_REASONING], n_src, n_rsn)
    finite = step().float()
    page, slot = int(caches.source.page_table[1, (n_src - 1) // 16]), (n_src - 1) % 16
    if fp8:
        caches.source.k_scale[page, :, slot] = float("nan")
    else:
        caches.source.k_pool[page, :, :, slot, :] = float("nan")       # (sequence 1, its last source token, every head)
    out = step().float()
    torch.cuda.synchronize()
    assert torch.isfinite(finite).all() and torch.equal(out[0], finite[0])
    assert torch.isnan(out[1]).all()
