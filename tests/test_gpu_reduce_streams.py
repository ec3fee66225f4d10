"""Accumulating reduces on several streams into one set of outputs: counts,
hash and XOR-fold of the pieces of a range, enqueued without any order between
the streams, against one reduce of the whole range.  Integers: results are
equal or wrong.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import grid_instance, low_rank_symmetric
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu

pytestmark = pytest.mark.gpu

STREAMS, PIECES = 8, 256


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("n,rank,total", [(36, 36, 1 << 16), (100, 20, 50001), (1024, 20, (1 << 14) + 77)])
def test_concurrent_accumulation(n, rank, total):
    A = grid_instance(6, b="1" * 36) if n == 36 else low_rank_symmetric(n, rank, 5)
    F, st = gpu_factor(A)
    assert st == hlf.HLF_OK and (1 << int(F.rank.item())) >= total
    want = hlf.enumerate_reduce(F, 0, total)
    counts, h, x = (torch.zeros_like(t) for t in want)
    cuts = np.linspace(0, total, PIECES + 1).astype(int)
    streams = [torch.cuda.Stream() for _ in range(STREAMS)]
    torch.cuda.synchronize()
    for k in range(PIECES):
        hlf.enumerate_reduce(F, int(cuts[k]), int(cuts[k + 1] - cuts[k]), accumulate=True, counts=counts,
                             hash_out=h, xorfold=x, stream=streams[k % STREAMS])
    torch.cuda.synchronize()
    assert torch.equal(h, want[1])
    assert torch.equal(counts, want[0])
    assert torch.equal(x, want[2])
