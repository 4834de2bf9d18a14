"""GPU, bf16: results that are written over inputs.  Rows of other workgroups are still to be read from those, so such calls work on packed copies;
what they give is what separate buffers give."""
import numpy as np
import pytest
import torch

import workloads as W

from gpu_helpers import DEV, ids_to_dev, to_dev

pytestmark = pytest.mark.gpu

LISTS = [(np.array([300, 41]), np.array([200, 77])), (np.array([1]), np.array([130])), (np.array([64, 400]), np.array([0, 65]))]


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


def _case(st, hq, hkv, d):
    cfg = W._assemble("shared", "bf16", hq, hkv, d, LISTS, "interleaved", 91)
    x = dict(zip("qkv", (to_dev(t, "bf16") for t in cfg.tensors())))
    x["d_out"] = to_dev(W.normal(np.random.Generator(np.random.PCG64(92)), tuple(x["q"].shape), "bf16"), "bf16")
    return cfg, x, st.st_plan_create(*ids_to_dev(cfg), cfg.cu_seqlens)


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("hq,hkv,d", [(3, 3, 64), (2, 2, 128), (6, 2, 64), (8, 2, 128)])
@pytest.mark.parametrize("over", ["q", "k", "v", "middle of v"])
def test_forward_output_over_an_input(st, hq, hkv, d, fused, over):
    cfg, x, plan = _case(st, hq, hkv, d)
    positions = torch.from_numpy(cfg.positions).to(DEV)
    run = lambda q, k, v, **kw: (st.st_attn_prefill_rope(q, k, v, positions, cfg.theta, plan, **kw) if fused else st.st_attn_prefill(q, k, v, plan, **kw))
    want = run(x["q"], x["k"], x["v"])
    n, size = cfg.n_tokens, x["q"].numel()
    flat = torch.zeros(2 * size, dtype=torch.bfloat16, device=DEV)
    out = flat[:size].view(n, hq, d)
    name = over[-1]
    at = size - 64 * d if over == "middle of v" else 0             # (the input begins among the last rows of the output)
    ins = {c: x[c].clone() for c in "qkv"}
    ins[name] = flat[at:at + x[name].numel()].view(x[name].shape)
    ins[name].copy_(x[name])
    got = run(ins["q"], ins["k"], ins["v"], out=out)
    assert torch.equal(got, want)


# (what lies at which element of one buffer; the others have buffers of their own)
@pytest.mark.parametrize("shared", [("dq", "q", 0), ("dq", "d_out", 0), ("dq", "out", 0), ("dq", "out", 1024), ("dk", "q", 0), ("dv", "d_out", 64), ("dk", "k", 0),
                                    ("dv", "v", 0), ("dk", "out", 0)])
@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 64), (3, 3, 128), (8, 2, 128), (4, 1, 64)])
@pytest.mark.parametrize("shift", [0, 1])
def test_gradients_over_an_input(st, hq, hkv, d, shared, shift):
    """shift 1: every tensor begins behind a 16-byte boundary."""
    cfg, x, plan = _case(st, hq, hkv, d)
    lse = torch.empty((cfg.n_tokens, hq), dtype=torch.float32, device=DEV)
    x["out"] = st.st_attn_prefill(x["q"], x["k"], x["v"], plan, lse=lse)
    want = dict(zip(("dq", "dk", "dv"), st.st_attn_prefill_bwd(x["d_out"], x["q"], x["k"], x["v"], x["out"], lse, plan)))
    grad, name, at = shared
    shapes = {**{c: t.shape for c, t in x.items()}, **{c: t.shape for c, t in want.items()}}
    buf = {c: torch.full((s.numel() + 2048 + shift,), float("nan"), dtype=torch.bfloat16, device=DEV) for c, s in shapes.items()}
    view = {c: buf[c][shift:shift + s.numel()].view(s) for c, s in shapes.items()}
    view[grad] = buf[name][shift + at:][:shapes[grad].numel()].view(shapes[grad])
    for c, t in x.items():
        view[c].copy_(t)
    lib = st.load_library()
    ws = torch.empty(int(lib.st_prefill_bwd_workspace_bytes(plan.handle, hq, hkv, d, st.ST_BF16)), dtype=torch.uint8, device=DEV)
    status = lib.st_attn_prefill_bwd(*(view[c].data_ptr() for c in ("dq", "dk", "dv", "d_out", "q", "k", "v", "out")), lse.data_ptr(), plan.handle, hq, hkv,
                                     d, 0.0, st.ST_BF16, ws.data_ptr(), ws.nbytes, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert status == 0
    for c in want:
        assert torch.equal(view[c], want[c]), c


@pytest.mark.parametrize("at", [0, 1024])
def test_gradient_over_the_output_while_kernels_are_timed(st, at):
    """Timed kernels are launched several times: the second launch must not read an output that the first has written over."""
    cfg, x, plan = _case(st, 4, 2, 128)
    lse = torch.empty((cfg.n_tokens, 4), dtype=torch.float32, device=DEV)
    out = st.st_attn_prefill(x["q"], x["k"], x["v"], plan, lse=lse)
    want = st.st_attn_prefill_bwd(x["d_out"], x["q"], x["k"], x["v"], out, lse, plan)
    flat = torch.zeros(2 * out.numel(), dtype=torch.bfloat16, device=DEV)
    view = flat[at:at + out.numel()].view(out.shape)
    view.copy_(out)
    dq, dk, dv = flat[:out.numel()].view(out.shape), torch.empty_like(x["k"]), torch.empty_like(x["v"])
    lib = st.load_library()
    ws = torch.empty(int(lib.st_prefill_bwd_workspace_bytes(plan.handle, 4, 2, 128, st.ST_BF16)), dtype=torch.uint8, device=DEV)
    st.st_profile_repeat(4)
    st.st_profile_enable(True)
    try:
        status = lib.st_attn_prefill_bwd(*(t.data_ptr() for t in (dq, dk, dv, x["d_out"], x["q"], x["k"], x["v"], view)), lse.data_ptr(), plan.handle, 4, 2,
                                         128, 0.0, st.ST_BF16, ws.data_ptr(), ws.nbytes, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        for which in (st.ST_PROF_BWD_DQ, st.ST_PROF_BWD_DKV):
            st.st_profile_read(which)
        st.st_profile_enable(False)
        st.st_profile_repeat(1)
    assert status == 0
    for got, ref in zip((dq, dk, dv), want):
        assert torch.equal(got, ref)
