"""Membership with many strings: waves take several blocks of 64 strings each
(a workgroup has 8 or 12 waves and, at 2^18 strings, 16 blocks on 256 compute
units), and from n = 576 on more kernel vectors than one group holds make every
block come round again, mostly to another wave than the one that wrote its
flags.  Every flag against K z = K l (mod 2) with the oracle's kernel basis K
and shift l.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import low_rank_symmetric
from oracle import hlf_oracle as O
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu
from test_gpu_membership_blocks import _bits, _words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# n, n - r: one group (12 and 8 waves), two to four groups
CASES = [(250, 100), (420, 419), (600, 600), (832, 500), (1000, 260), (1024, 257), (1024, 600), (1024, 1024)]


@pytest.mark.parametrize("n,nk", CASES)
def test_every_flag(n, nk):
    A = low_rank_symmetric(n, n - nk, n + nk) if nk < n else np.zeros((n, n), dtype=np.uint8)
    Fo = O.factor(A)
    got = n - Fo["rank"]
    F, st = gpu_factor(A)
    assert st == hlf.HLF_OK and abs(got - nk) <= 1
    W = hlf.words_for(n)
    K, l = _bits(Fo["kernel"][:got], n), _bits([Fo["shift"]], n)
    B = _bits(Fo["basis"], n) if Fo["rank"] else np.zeros((0, n), np.uint8)
    rng = np.random.default_rng(n * 3000 + nk)
    # exact ones; one bit flipped at a free column of the first, the middle and
    # the last kernel vectors; uniform ones
    k = 4096
    z = (rng.integers(0, 2, (k, B.shape[0])).astype(np.float32) @ B.astype(np.float32)).astype(np.int64).astype(np.uint8) & 1
    z ^= l
    free = [int(np.nonzero(v)[0][-1]) for v in K]
    for part, vectors in ((2, free[:3]), (3, free[got // 2 : got // 2 + 3]), (4, free[-3:])):
        rows = np.arange(part * k // 8, (part + 1) * k // 8)
        z[rows, rng.choice(vectors, rows.size)] ^= 1
    z[7 * k // 8 :] = rng.integers(0, 2, (k // 8, n))
    want = ((((z ^ l).astype(np.float32) @ K.T.astype(np.float32)).astype(np.int64) & 1).sum(axis=1) == 0).astype(np.uint8)
    words = torch.from_numpy(_words(z, W)).cuda()
    bad, late = np.nonzero(want == 0)[0], np.arange(4 * k // 8, 5 * k // 8)
    for num in (1 << 18, (1 << 18) + (1 << 17) + 37):
        pick = rng.integers(0, k, num)
        pick[: num // 8] = rng.choice(bad, num // 8)  # blocks that fail as a whole, some in the last group only
        pick[num // 8 : num // 4] = rng.choice(late, num // 4 - num // 8)
        print(f"[member] n={n} n-r={got} strings={num}", flush=True)
        strings = words[torch.from_numpy(pick).cuda()].contiguous()
        out = torch.full((num + 8,), 9, dtype=torch.uint8, device="cuda")
        hlf.membership(F, strings, out=out[:num])
        res = out.cpu().numpy()
        assert np.array_equal(res[:num], want[pick]), (n, nk, num)
        assert (res[num:] == 9).all()
