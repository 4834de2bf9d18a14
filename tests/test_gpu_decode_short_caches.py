"""GPU: decode over short caches on both sides of the line between one launch (a workgroup finishes the rows of a sequence and KV
head itself) and the split with its merge: the bound one short of, at and one past the line, 40, 41 and more than 256 workgroups --
against the fp64 oracle, with the bounds of the parity suite."""
import numpy as np
import pytest
import torch

from test_gpu_decode_long_units import _stamped_workgroups
from test_gpu_parity import _check_decode

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


@pytest.mark.parametrize("batch,hq,hkv,d,line", [(5, 16, 8, 128, 832), (41, 2, 1, 128, 1024), (1, 4, 2, 64, 1024), (33, 16, 8, 64, 1024), (33, 32, 8, 128, 1024)])
@pytest.mark.parametrize("past", [-1, 0, 1])
def test_line_between_one_launch_and_the_split(st, batch, hq, hkv, d, line, past):
    rng = np.random.Generator(np.random.PCG64(470 + batch))
    src_lens = rng.integers(0, 200, batch); rsn_lens = rng.integers(1, 200, batch)
    src_lens[0] = 300; rsn_lens[0] = line + past - 300                          # the bounds are the longest caches
    src_vis = np.minimum(src_lens, rng.integers(0, 400, batch)); src_vis[0] = 300
    (caches, tq, out), stamped = _stamped_workgroups(st, lambda: _check_decode(st, rng, batch, hq, hkv, d, src_lens, rsn_lens, src_vis))
    assert (stamped > 0) == (past > 0)                                           # (only the split kernel leaves stamps)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("q_len,hq,hkv", [(1, 8, 8), (1, 32, 8), (2, 16, 2), (4, 32, 8)])
def test_more_short_caches_than_compute_units(st, q_len, hq, hkv, d):
    """Two workgroups on a compute unit and a second round of them: rows 1 to 16, empty caches, one token, a step that ends in a page."""
    rng = np.random.Generator(np.random.PCG64(480 + q_len + d))
    batch = 530 // hkv
    src_lens = rng.choice([0, 1, 17, 64, 129], batch); rsn_lens = rng.choice([q_len, 5, 31, 33, 64, 200], batch)
    _check_decode(st, rng, batch, hq, hkv, d, src_lens, rsn_lens, np.minimum(src_lens, rng.integers(0, 140, batch)), q_len=q_len, rope_theta=1.0e6)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("q_len,hq,hkv", [(1, 7, 1), (1, 9, 1), (3, 3, 1), (5, 1, 1), (3, 10, 2), (13, 1, 1)])
def test_rows_that_fill_the_merge_in_part(st, q_len, hq, hkv, d):
    """3 to 15 rows: the merge takes one, two or four dims of a row per thread, the last threads none; an empty and a one-token cache."""
    rng = np.random.Generator(np.random.PCG64(490 + q_len * hq + d))
    src_lens, rsn_lens = np.array([0, 70, 33]), np.array([q_len, q_len + 1, 200])
    _check_decode(st, rng, 3, hq, hkv, d, src_lens, rsn_lens, np.minimum(src_lens, 64), q_len=q_len, rope_theta=1.0e6)
