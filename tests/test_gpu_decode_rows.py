"""GPU: the decode step with 17 to 32 query rows per sequence and KV head (several tokens in one call, wide groups), over
every work-unit size, both head sizes, ragged and empty caches, with and without the fused rotation -- against the fp64
oracle, with the bounds of the parity suite."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import streaming_attention as O

from gpu_helpers import DEV, to_dev, to_f64
from test_gpu_parity import _check_decode, _fill_dual

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


@pytest.mark.parametrize("unit", [0, 128, 512, 1024])
@pytest.mark.parametrize("q_len,hq,hkv,d,rope", [(17, 1, 1, 128, None), (8, 8, 2, 128, 1.0e6), (5, 4, 1, 64, 1.0e6), (1, 32, 1, 128, None)])
def test_decode_17_to_32_rows(st, unit, q_len, hq, hkv, d, rope):
    rng = np.random.Generator(np.random.PCG64(450 + q_len + unit))
    # units cut exactly, one short and one past; steps of 32 tokens with one token in them; nothing visible in the source
    src_lens = np.array([1100, 129, 640, 31, 33]); rsn_lens = np.array([700, 1500, 127, 1025, 32])
    src_vis = np.array([1025, 128, 0, 31, 33])
    _check_decode(st, rng, 5, hq, hkv, d, src_lens, rsn_lens, src_vis, q_len=q_len, rope_theta=rope, unit_tokens=unit)


@pytest.mark.parametrize("q_len,hq,hkv,d", [(1, 2, 1, 128), (8, 8, 2, 128), (2, 16, 2, 64)])
def test_decode_rows_of_many_partials(st, q_len, hq, hkv, d):
    """The merge of a row's partial results over one to eight groups of a workgroup, in one and in several round trips: 128-token
    units of caches with one, eight, nine and about a hundred of them; a source slice that ends in the first unit."""
    rng = np.random.Generator(np.random.PCG64(460 + q_len))
    for src_lens, rsn_lens in ((np.array([130]), np.array([128 * 6])), (np.array([9000, 100]), np.array([4100, 40])), (np.array([1200]), np.array([9]))):
        src_vis = np.minimum(src_lens, np.arange(9000, 0, -8900)[:len(src_lens)])
        _check_decode(st, rng, len(src_lens), hq, hkv, d, src_lens, rsn_lens, src_vis, q_len=q_len, unit_tokens=128)


@pytest.mark.parametrize("d", [64, 128])
def test_precision_of_17_to_32_rows(st, d):
    """Error of the rows in the 2-norm, N(0, 1) inputs: the rounding of the results (2^-7 / sqrt(12) of a power of two, 0.735 of it
    over values spread evenly in the logarithm: 1.66e-3), that of the weights (1.10e-3 where the largest of 32 tokens is 1, which is
    exact; 1.60e-3 with any other reference) -- together 1.99e-3, or 2.31e-3.  The bound lies between the two; a running maximum over
    512 tokens gives 2.10e-3."""
    rng = np.random.Generator(np.random.PCG64(470 + d))
    src, rsn = rng.integers(300, 3000, 8), rng.integers(300, 3000, 8)
    caches, ref, _ = _fill_dual(st, rng, 8, 2, d, src, rsn)
    q = W.normal(rng, (8, 8, 8, d), "bf16")
    ts, tr = (torch.from_numpy(x.astype(np.int32)).to(DEV) for x in (src, rsn))
    out = st.st_attn_decode_dual(to_dev(q, "bf16"), caches, ts, tr, int(src.max()), int(rsn.max()))
    num = den = 0.0
    for b in range(8):
        o_ref, _ = O.decode_dual_concat(q[b].astype(np.float64), *[ref[w][i][b] for w in (st.ST_SOURCE, st.ST_REASONING) for i in (0, 1)], int(src[b]), int(rsn[b]))
        num += ((to_f64(out[b]) - o_ref) ** 2).sum()
        den += (o_ref ** 2).sum()
    assert (num / den) ** 0.5 <= 2.1e-3


def test_scores_that_fall_for_long(st):
    """Scores that fall by hundreds of octaves from one step of a wave to the next: the reference may not follow them all the way."""
    caches, ref, _ = _fill_dual(st, np.random.Generator(np.random.PCG64(480)), 1, 1, 64, np.array([4000]), np.array([1500]))
    for cache, n in ((caches.source, 4000), (caches.reasoning, 1500)):
        k = torch.zeros((cache.n_pages, 16, 1, 64), dtype=torch.bfloat16, device=DEV)
        table = cache.page_table[0].long()
        rows = torch.zeros((table.numel() * 16, 64), dtype=torch.float32, device=DEV)
        rows[:n, 0] = -2.0 * torch.arange(n, device=DEV)
        k[table] = rows.to(torch.bfloat16).view(-1, 16, 1, 64)
        cache.k_pool.copy_(st.k_pool_from_logical(k))
    q = torch.zeros((1, 20, 1, 64), dtype=torch.bfloat16, device=DEV)
    q[..., 0] = 8.0                                               # scores of 0, -2, -4 ... with the scale of 1 / 8
    lens = [torch.tensor([n], dtype=torch.int32, device=DEV) for n in (4000, 1500)]
    lse = torch.empty((1, 20, 1), dtype=torch.float32, device=DEV)
    out = st.st_attn_decode_dual(q, caches, *lens, 4000, 1500, lse=lse, unit_tokens=1024)
    w = np.exp(np.arange(0.0, -40.0, -2.0))                       # keys rounded to bf16: the first 128 of them exactly
    v = [ref[w_][1][0].astype(np.float64) for w_ in (st.ST_SOURCE, st.ST_REASONING)]
    expect = sum(w @ x[:20, 0] for x in v) / (2 * w.sum())
    assert np.abs(to_f64(out[0, :, 0]) - expect).max() <= 2e-2
    assert np.abs(to_f64(lse[0, :, 0]) - np.log(2 * w.sum())).max() <= 1e-3


@pytest.mark.parametrize("units", [2, 4, 6, 8, 12, 16])
@pytest.mark.parametrize("q_len,hq,hkv,d,fp8", [(1, 4, 2, 128, False), (8, 8, 2, 64, False), (2, 8, 2, 128, True)])
def test_units_of_a_head_in_turn(st, units, q_len, hq, hkv, d, fp8):
    """Unit counts that share a factor with the eight XCDs: the units of a head then begin at another one from head to head.  Every
    unit of every head is still taken once: eleven sequences, one of them full, the others of a unit or two."""
    rng = np.random.Generator(np.random.PCG64(490 + units))
    src, rsn = rng.integers(1, 200, 11), rng.integers(q_len, 200, 11)
    src[3], rsn[3] = 128, 128 * (units - 1)
    src = np.minimum(src, 128)                                     # one unit of the source, the others of the reasoning cache
    rsn = np.minimum(rsn, 128 * (units - 1))
    _check_decode(st, rng, 11, hq, hkv, d, src, rsn, src, q_len=q_len, fp8=fp8, unit_tokens=128)
