"""GPU: the decode step with 17 to 32 query rows per sequence and KV head (several tokens in one call, wide groups), over
every work-unit size, both head sizes, ragged and empty caches, with and without the fused rotation -- against the fp64
oracle, with the bounds of the parity suite."""
import numpy as np
import pytest
import torch

from test_gpu_parity import _check_decode

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
