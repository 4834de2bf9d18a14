"""GPU: gradients from and into tensors that are only aligned to their elements (slices of a flat buffer) are bit for bit those of
16-byte aligned ones."""
import numpy as np
import pytest
import torch

import workloads as W

from gpu_helpers import DEV, ids_to_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


def _shifted(t, elements):
    """A copy of t that begins `elements` elements behind a 16-byte boundary."""
    flat = torch.zeros(t.numel() + 16, dtype=t.dtype, device=t.device)
    view = flat[elements:elements + t.numel()].view(t.shape)
    view.copy_(t)
    assert view.data_ptr() % 16 == elements * t.element_size()
    return view


# (the last two split the query heads of a group: the sums of the parts are stored by a kernel of their own)
@pytest.mark.parametrize("dtype,shift,hq,hkv,d,lists", [
    ("f32", 1, 4, 2, 64, [([30, 40], [25, 50])]), ("f32", 3, 2, 2, 128, [([70], [33])]), ("bf16", 1, 4, 2, 128, [([30, 40], [25, 50])]),
    ("bf16", 6, 2, 1, 64, [([70], [133])]), ("f32", 2, 8, 2, 64, [([40], [50])]), ("bf16", 3, 8, 1, 64, [([300], [400])])])
def test_gradients_of_slices(st, dtype, shift, hq, hkv, d, lists):
    cfg = W._assemble("slices", dtype, hq, hkv, d, [tuple(map(np.array, x)) for x in lists], "interleaved", 51)
    q, k, v = (to_dev(x, dtype) for x in cfg.tensors())
    g = to_dev(W.normal(np.random.Generator(np.random.PCG64(52)), tuple(q.shape), dtype), dtype)
    plan = st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)
    lse = torch.empty((cfg.n_tokens, hq), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(q, k, v, plan, lse=lse)
    want = st.st_attn_prefill_bwd(g, q, k, v, out, lse, plan)
    lib, code = st.load_library(), st.ST_F32 if dtype == "f32" else st.ST_BF16
    grads = [_shifted(torch.full_like(x, float("nan")), shift) for x in (q, k, v)]
    ins = [_shifted(x, shift) for x in (g, q, k, v, out)]
    ws = torch.empty(int(lib.st_prefill_bwd_workspace_bytes(plan.handle, hq, hkv, d, code)), dtype=torch.uint8, device=DEV)
    status = lib.st_attn_prefill_bwd(*(x.data_ptr() for x in (*grads, *ins)), lse.data_ptr(), plan.handle, hq, hkv, d, 0.0, code,
                                     ws.data_ptr(), ws.nbytes, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert status == 0
    for name, got, ref in zip(("dq", "dk", "dv"), grads, want):
        assert torch.equal(got, ref), name
