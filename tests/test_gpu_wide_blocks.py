"""Multi-word windows at the edges of the launch rule: from one tile per
workgroup to kWideFill of them in one generation of two workgroups per compute
unit, and past that, in both orders and from odd indices (in counter order the
step from tile to tile is the carry's rows).  Against the kernel for unaligned
outputs, which looks every solution up by itself, and the oracle at the ends.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import low_rank_symmetric
from oracle import c_oracle as C
from oracle import hlf_oracle as O
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu

pytestmark = pytest.mark.gpu

FILL = 32  # most tiles per workgroup in one generation


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("n", [100, 180, 250, 300, 512, 570, 1000])
def test_launch_edges(n):
    A = low_rank_symmetric(n, 24, 3)
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    W = hlf.words_for(n)
    tile = 256 if W <= 4 else 128 if W <= 8 else 64
    blocks = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    edges = [blocks, 2 * blocks, 3 * blocks, FILL * blocks]
    cases = [(b, t * tile + d) for t in edges for b, d in ((0, 0), (0, 1), (3 * tile - 5, -tile), (5, 7))]
    top = 1 << Fo["rank"]
    most = max(c for _, c in cases)
    assert most + 3 * tile <= top
    buf = torch.empty(8 * W * most + 32, dtype=torch.uint8, device="cuda")
    for flags, ref in ((0, C.enumerate_range), (hlf.HLF_ORDER_COUNTER, C.enumerate_counter_range)):
        for begin, count in cases:
            print(f"[wide] {W} words, begin {begin}, count {count}, flags {flags}", flush=True)
            out = torch.full((count + 2, W), 7, dtype=torch.int64, device="cuda")
            st = hlf.lib().hlf_enumerate_ex(F.c, begin, count, 64 * W, flags, out[1:].data_ptr(), hlf._stream())
            assert st == hlf.HLF_OK
            assert bool((out[0] == 7).all()) and bool((out[-1] == 7).all())
            st = hlf.lib().hlf_enumerate_ex(F.c, begin, count, 64 * W, flags, buf.data_ptr() + 1, hlf._stream())
            assert st == hlf.HLF_OK
            want = buf[1 : 1 + 8 * W * count]
            assert torch.equal(out[1:-1].reshape(-1).view(torch.uint8), want)
            for b, c in ((begin, 65), (begin + count - 65, 65)):
                got = out[1 + b - begin : 1 + b - begin + c].cpu().numpy().view(np.uint64)
                assert np.array_equal(got, ref(Fo, b, c))
    assert int(F.status.item()) == hlf.HLF_OK
