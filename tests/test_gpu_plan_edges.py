"""GPU: the segment-table builder at the edges of its chunks and of its two ways of taking the offsets -- sequences one token
short of, exactly and one past 1,024 and 16,384 tokens (what a thread keeps in registers), source streams around 8,192 tokens
(what is searched in LDS), batches around 64 and 512 -- bit-exact against the oracle's metadata."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_parity import _check_metadata

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def st():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2510_17238_amd as st_
    st_.load_library()
    return st_


def _lengths(total, n_src, pieces):
    """Source and reasoning segments of one sequence of `total` tokens with `n_src` source tokens in `pieces` segments."""
    cut = lambda n: np.diff(np.linspace(0, n, pieces + 1).astype(np.int64))
    return cut(n_src), cut(total - n_src)


@pytest.mark.parametrize("layout,sizes", [("interleaved", [(1023, 400, 7), (1024, 1, 1), (1025, 1024, 9), (1, 0, 1), (4097, 2000, 33)]),
                                          ("grouped", [(16383, 8191, 40), (900, 300, 5)]),
                                          ("interleaved", [(16385, 8192, 40), (16384, 100, 3)]),
                                          ("interleaved", [(17500, 8300, 50)])])
def test_plan_chunk_edges(st, layout, sizes):
    _check_metadata(st, W._assemble("plan-edges", "f32", 2, 1, 64, [_lengths(*x) for x in sizes], layout, 31))


@pytest.mark.parametrize("batch", [63, 64, 65, 511, 512, 513])
def test_plan_batch_edges(st, batch):
    rng = np.random.Generator(np.random.PCG64(32))
    lists = [W.draw_pairs(rng, 2, (0, 4), (0, 5)) for _ in range(batch)]
    _check_metadata(st, W._assemble("plan-batches", "f32", 2, 1, 64, lists, "interleaved", 33))
