"""hlf_solve_dense around the sizes where its grid changes: blocks of at most
128 KiB, one generation of workgroups of 128 to 512 KiB, blocks again.  Against
hlf_enumerate of the record it wrote, which takes another kernel.
"""

import pytest
import torch

from hlf_inputs import grid_instance
from paper_2103_00693_amd import hlf

from gpu_util import device_matrix, require_gpu

pytestmark = pytest.mark.gpu

DTYPES = {32: torch.int32, 64: torch.int64}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("tiles_per_block", [1, 7, 8, 32, 33])
def test_grid_edges(bits, tiles_per_block):
    N = 5 if bits == 32 else 6
    A = device_matrix(grid_instance(N, b="1" * (N * N)))
    F = hlf.Factors(N * N)
    V = 128 // bits
    blocks = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    edge = 1024 * V * blocks * tiles_per_block  # the most solutions at that many tiles each
    hlf.solve_dense(A, F, 0, 0, bits)
    top = 1 << int(F.rank.item())
    for begin, count in ((0, edge), (0, edge + 1), (V, edge - V - 1), (3 * V, edge + 1024 * V)):
        count = min(count, top - begin)
        print(f"[solve] {bits} bits, begin {begin}, count {count}", flush=True)
        out = torch.full((count + 8,), 7, dtype=DTYPES[bits], device="cuda")
        hlf.solve_dense(A, F, begin, count, bits, out=out[:count])
        want = hlf.enumerate_solutions(F, begin, count, bits)
        assert int(F.status.item()) == hlf.HLF_OK
        assert torch.equal(out[:count], want) and bool((out[count:] == 7).all())
