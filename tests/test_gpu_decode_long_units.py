"""GPU: the work units of 2,048 and 4,096 tokens, which only large launches take (they cannot be pinned) -- many sequences over the
pages of a few, so that the launch is large and the caches are small; against the fp64 oracle, with the bounds of the parity
suite.  And the rule that chooses the unit: the number of workgroups that a launch stamps."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import streaming_attention as O

from gpu_helpers import DEV, to_dev, to_f64
from test_gpu_parity import _fill_dual

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


def _stamped_workgroups(st, step):
    """Runs `step` with the wave timeline on; (its result, workgroups of the split kernel's launch)."""
    buf = torch.zeros((1 << 16, 2), dtype=torch.int64, device=DEV)
    st.st_profile_wave_trace(buf)
    st.st_profile_enable(True)
    try:
        out = step()
    finally:
        st.st_profile_enable(False)
        st.st_profile_wave_trace(None)
    torch.cuda.synchronize()
    st.st_profile_read(st.ST_PROF_DECODE_SPLIT)
    return out, int((buf[:, 1] > 0).sum())


def _many_over_few(st, caches, copies, bound, hkv, d, fp8):
    """The few sequences of `caches`, `copies` times over, with page tables for `bound` tokens (pages past a sequence's own: any)."""
    wide = []
    for c in (caches.source, caches.reasoning):
        table = torch.zeros((c.batch, bound // 16), dtype=torch.int32, device=DEV)
        own = min(c.max_pages_per_seq, bound // 16)
        table[:, :own] = c.page_table[:, :own]
        w = st.KVCache(1, copies * c.batch, bound // 16, hkv, d, table.repeat(copies, 1).contiguous(), fp8=fp8)
        w.n_pages, w.k_pool, w.v_pool, w.k_scale, w.v_scale = c.n_pages, c.k_pool, c.v_pool, c.k_scale, c.v_scale
        wide.append(w)
    return st.DualCache(*wide)


# lengths one short of, at and one past a unit of 4,096 (bound 8,192) or 2,048 tokens (bound 4,096), full caches, one token, none
LENS = {8192: (np.array([4095, 4097, 8192, 0]), np.array([8191, 4096, 33, 4097])), 4096: (np.array([2047, 2049, 4096, 0]), np.array([4095, 2048, 33, 2049]))}


@pytest.mark.parametrize("bound,unit", [(8192, 4096), (4096, 2048)])
@pytest.mark.parametrize("q_len,hq,d,rope,fp8,copies", [(1, 2, 128, None, False, 64), (4, 4, 64, 1.0e6, False, 64), (4, 8, 128, 1.0e6, False, 12),
                                                        (8, 4, 64, None, False, 12), (1, 4, 128, None, True, 24), (4, 8, 64, 1.0e6, True, 24)])
def test_long_units(st, bound, unit, q_len, hq, d, rope, fp8, copies):
    _check_long_units(st, bound, unit, q_len, hq, d, rope, fp8, copies)


@pytest.mark.parametrize("q_len,hq,d,rope", [(8, 8, 128, 1.0e6), (5, 8, 64, None)])
def test_longest_units_with_17_to_32_rows(st, q_len, hq, d, rope):
    _check_long_units(st, 8192, 4096, q_len, hq, d, rope, False, 6)


def _check_long_units(st, bound, unit, q_len, hq, d, rope, fp8, copies):
    rng = np.random.Generator(np.random.PCG64(490 + q_len))
    hkv, (src, rsn) = 2, LENS[bound]
    few, ref, _ = _fill_dual(st, rng, 4, hkv, d, src, rsn, chunks=(2048,), rope_theta=None if fp8 else rope, fp8=fp8,
                             row_exponents=(-4, 1) if fp8 else None)
    caches = _many_over_few(st, few, copies, bound, hkv, d, fp8)
    q = W.normal(rng, (4, q_len, hq, d), "bf16")
    tq = to_dev(q, "bf16").repeat(copies, 1, 1, 1)
    ts, tr = (torch.from_numpy(np.tile(x, copies).astype(np.int32)).to(DEV) for x in (src, rsn))
    lse = torch.empty((4 * copies, q_len, hq), dtype=torch.float32, device=DEV)
    step = lambda: st.st_attn_decode_dual(tq, caches, ts, tr, bound, bound, lse=lse, rope_theta=rope)
    out, workgroups = _stamped_workgroups(st, step)
    if not fp8 and q_len * hq <= 16 * hkv:                    # (the kernel that leaves stamps)
        assert workgroups == 4 * copies * hkv * 2 * (bound // unit)
    assert torch.equal(out.view(copies, -1), out[:4].reshape(1, -1).expand(copies, -1))      # every copy gives the same rows
    for b in range(4):
        args = [ref[w][i][b] for w in (st.ST_SOURCE, st.ST_REASONING) for i in (0, 1)] + [int(src[b]), int(rsn[b])]
        qb = q[b].astype(np.float64)
        if rope is not None:
            qb = O.rope(qb, int(rsn[b]) - q_len + np.arange(q_len), rope)
        o_ref, l_ref = (O.decode_dual_fp8 if fp8 else O.decode_dual_concat)(qb, *args)
        assert np.abs(to_f64(out[b]) - o_ref).max() <= 2e-2 * (max(1.0, np.abs(o_ref).max()) if fp8 else 1.0), b
        assert np.abs(to_f64(lse[b]) - l_ref).max() <= 2e-2, b


@pytest.mark.parametrize("batch,q_len,hq,src,rsn,units", [(64, 1, 8, 5000, 5000, 5 + 5), (64, 1, 8, 8192, 8192, 2 + 2), (20, 4, 32, 3000, 900, 3 + 1),
                                                          (20, 4, 32, 4096, 4096, 2 + 2), (64, 1, 8, 500, 6000, 1 + 6), (64, 4, 32, 700, 700, 1 + 1)])
def test_unit_leaves_no_long_and_short_workgroups(st, batch, q_len, hq, src, rsn, units):
    """Units per sequence and KV head: a unit that the caches fill, not one that leaves a long and a short workgroup of each."""
    hkv, d = 8, 64
    caches = []
    for n in (src, rsn):
        pages = (n + 15) // 16
        caches.append(st.KVCache(pages, batch, pages, hkv, d, torch.arange(pages, dtype=torch.int32, device=DEV).repeat(batch, 1), fill=0.5))
    tq = torch.ones((batch, q_len, hq, d), dtype=torch.bfloat16, device=DEV)
    lens = [torch.full((batch,), n, dtype=torch.int32, device=DEV) for n in (src, rsn)]
    step = lambda: st.st_attn_decode_dual(tq, st.DualCache(*caches), *lens, src, rsn)
    out, workgroups = _stamped_workgroups(st, step)
    assert workgroups == batch * hkv * units
    assert torch.equal(out, torch.full_like(out, 0.5))        # (equal scores over equal values)
