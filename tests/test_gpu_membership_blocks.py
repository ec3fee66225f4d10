"""The matrix-core membership kernel (n > 192) at its edges, every flag against
K z = K l (mod 2) with the oracle's kernel basis K and shift l.

A wave takes 64 strings and the kernel vectors come in 32-chunks: an odd chunk
first, then pairs, in groups of at most 16 KiB of chunks times words.  The
instances have every word count, n - r around the chunk, pair and group edges
(up to n itself); the string counts are around the block edges and enough for
waves to take several blocks; strings start at any multiple of 8 bytes.
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


def _bits(ints, n):
    raw = np.array([np.frombuffer(int(v).to_bytes((n + 7) // 8, "little"), dtype=np.uint8) for v in ints])
    return np.unpackbits(raw.reshape(len(ints), -1), axis=1, bitorder="little")[:, :n]


def _words(bits, W):
    pad = np.zeros((bits.shape[0], 64 * W), dtype=np.uint8)
    pad[:, : bits.shape[1]] = bits
    return np.packbits(pad, axis=1, bitorder="little").view(np.int64)


CASES = [  # n, n - r
    (193, 1), (200, 33), (256, 32), (256, 256), (257, 64), (320, 65), (321, 96), (384, 97), (449, 128), (512, 130),
    (513, 160), (575, 575), (640, 192), (700, 224), (704, 225), (769, 256), (832, 289), (960, 191), (1000, 260),
    (1024, 0), (1024, 95), (1024, 257), (1024, 600), (1024, 1024),
]


@pytest.mark.parametrize("n,nk", CASES)
def test_every_flag(n, nk):
    print(f"[member] n={n} n-r={nk}", flush=True)
    A = low_rank_symmetric(n, n - nk, n + nk) if nk < n else np.zeros((n, n), dtype=np.uint8)
    if nk == 0:
        A = np.eye(n, dtype=np.uint8)
    Fo = O.factor(A)
    got = n - Fo["rank"]
    F, st = gpu_factor(A)
    assert st == hlf.HLF_OK and abs(got - nk) <= 1
    W = hlf.words_for(n)
    K, l = _bits(Fo["kernel"][:got], n) if got else np.zeros((0, n), np.uint8), _bits([Fo["shift"]], n)
    B = _bits(Fo["basis"], n) if Fo["rank"] else np.zeros((0, n), np.uint8)
    rng = np.random.default_rng(n * 2000 + nk)
    # exact ones, some with one bit flipped anywhere, some only at the last kernel vector's free column, uniform ones
    most = 64 * 1500 + 5
    k = 4096
    z = (rng.integers(0, 2, (k, B.shape[0])).astype(np.float32) @ B.astype(np.float32)).astype(np.int64).astype(np.uint8) & 1
    z ^= l
    z[k // 4 : k // 2, :][np.arange(k // 4), rng.integers(0, n, k // 4)] ^= 1
    if got:
        z[k // 2 : 5 * k // 8, int(np.nonzero(K[-1])[0][-1])] ^= 1
    z[7 * k // 8 :] = rng.integers(0, 2, (k // 8, n))
    z = z[rng.permutation(k)]
    lead = z[:64].copy()
    z[:64] = rng.integers(0, 2, (64, n))  # a block that fails as a whole
    z[64:128] = lead
    want = ((((z ^ l).astype(np.float32) @ K.T.astype(np.float32)).astype(np.int64) & 1).sum(axis=1) == 0).astype(np.uint8)
    words = torch.from_numpy(_words(z, W)).cuda()
    big = words.repeat(most // k + 1, 1)
    for num, first in ((1, 0), (63, 3), (64, 1), (65, 64), (1000, 7), (k, 0), (most, 1)):
        out = torch.full((num,), 9, dtype=torch.uint8, device="cuda")
        hlf.membership(F, big[first : first + num], out=out)
        expect = np.resize(want, most + k)[first : first + num]
        assert np.array_equal(out.cpu().numpy(), expect), (n, nk, num, first)
