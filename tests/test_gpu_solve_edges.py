"""hlf_solve_dense at the edges of its one-generation grid, 128 and 512 KiB per
workgroup, with an instance whose rank leaves room on both sides of each for
32-bit words too (a 5 x 5 grid ends below the upper one).  Against
hlf_enumerate of the record it wrote, which takes another kernel.
"""

import pytest
import torch

from hlf_inputs import random_symmetric
from paper_2103_00693_amd import hlf

from gpu_util import device_matrix, require_gpu

pytestmark = pytest.mark.gpu

DTYPES = {32: torch.int32, 64: torch.int64}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("tiles_per_block", [7, 32])
def test_both_sides_of_an_edge(bits, tiles_per_block):
    n = 30
    A = device_matrix(random_symmetric(n, 2, 0.5))
    F = hlf.Factors(n)
    V = 128 // bits
    blocks = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    edge = 1024 * V * blocks * tiles_per_block  # the most solutions at that many tiles of 1024 V each
    hlf.solve_dense(A, F, 0, 0, bits)
    top = 1 << int(F.rank.item())
    assert edge + 2048 * V <= top  # nothing is clamped
    for begin, count in ((0, edge), (0, edge + 1), (V, edge - V - 1), (3 * V, edge + 1024 * V)):
        print(f"[solve] {bits} bits, {tiles_per_block} tiles, begin {begin}, count {count}", flush=True)
        out = torch.full((count + 8,), 7, dtype=DTYPES[bits], device="cuda")
        hlf.solve_dense(A, F, begin, count, bits, out=out[:count])
        want = hlf.enumerate_solutions(F, begin, count, bits)
        assert int(F.status.item()) == hlf.HLF_OK
        assert torch.equal(out[:count], want) and bool((out[count:] == 7).all())
