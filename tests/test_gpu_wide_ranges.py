"""Materialised solutions of 2 to 16 words: every word count, ranges that begin
and end anywhere in a tile, in both orders, at any multiple of 8 bytes, against
the definition, and nothing written beside the range.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import low_rank_symmetric
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu
from oracle import hlf_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("order", ["gray", "counter"])
@pytest.mark.parametrize("W", range(2, 17))
def test_ranges(W, order):
    n = 64 * W - (W * 7) % 64
    rank = 20 + W % 3
    A = low_rank_symmetric(n, rank, 5 * n)
    ref = O.factor(A)
    r = ref["rank"]
    F, st = gpu_factor(A)
    assert st == hlf.HLF_OK and rank - 1 <= r <= rank
    top = 1 << r
    to_words = lambda v: [(v >> (64 * w)) & ((1 << 64) - 1) for w in range(W)]  # noqa: E731
    B = np.array([to_words(b) for b in ref["basis"]], dtype=np.uint64)
    low = np.array(to_words(ref["shift"]), dtype=np.uint64)
    print(f"[wide] W={W} n={n} r={r} {order}", flush=True)
    ranges = [(0, 1), (0, 64), (1, 2), (63, 2), (64, 256), (255, 258), (127, 130), (5, 4099), (top - 1, 1),
              (top - 777, 777), (top // 2 - 3, 20011), (123456, 65536)]
    for lead in (0, 1):  # 16-byte aligned, and 8 bytes past that
        for begin, count in ranges:
            buf = torch.full((count * W + 8,), 7, dtype=torch.int64, device="cuda")
            at = 2 + (lead + (buf.data_ptr() >> 3)) % 2
            out = buf[at : at + count * W].view(count, W)
            hlf.enumerate_solutions(F, begin, count, 64 * W, out=out, order=order)
            got = buf.cpu().numpy()
            assert (got[:at] == 7).all() and (got[at + count * W :] == 7).all(), (begin, count, lead)
            i = np.arange(begin, begin + count, dtype=np.uint64)
            c = i ^ (i >> np.uint64(1)) if order == "gray" else i
            want = np.tile(low, (count, 1))
            for k in range(r):
                want ^= B[k] * ((c >> np.uint64(k)) & np.uint64(1))[:, None]
            assert np.array_equal(got[at : at + count * W].view(np.uint64).reshape(count, W), want), (begin, count, lead)
