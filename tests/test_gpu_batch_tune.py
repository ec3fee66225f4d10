"""The batch autotuner where several candidates come to the same launch: it
reports the largest chunk size of them, so what is chosen does not hang on the
noise of equal timings, and the stored default still takes the large max_rank
that the untuned default takes.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import grid_instance
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("count,max_rank", [(23, 9), (31, 12), (54, 16)])
def test_equal_launches_report_the_largest_chunk(count, max_rank):
    """So few solutions that every chunk size is cut to pieces of 2^12."""
    mats = [grid_instance(1 + i % 4, 1.0, i) for i in range(count)]
    B = hlf.Batch([A.shape[0] for A in mats])
    A_dev = B.dense_input(mats)
    best, ms = B.tune(A_dev, max_rank)
    print(f"[tune] {count} instances, max_rank {max_rank}: {best}, {ms} ms", flush=True)
    assert best.chunk_log2 == 22 and best.waves_per_cu in (2, 4, 8, 12) and ms > 0
    # count * 2^(50 - 22) < 2^40 chunks; at 2^14 solutions each they would not fit
    B.reduce(A_dev, 50)
    counts, hashes = B.reduce_results()
    for i, A in enumerate(mats):
        F, _ = gpu_factor(A)
        c, h, _ = hlf.enumerate_reduce(F, 0, 1 << int(F.rank.item()))
        assert np.array_equal(counts[i], c.cpu().numpy().view(np.uint64))
        assert hashes[i] == int(h.item()) & ((1 << 64) - 1)
