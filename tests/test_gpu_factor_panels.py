"""Stage 1's 64-column panels at their edges, bit for bit against the oracle.

The workgroup kernel finds a panel's pivots in batches of 64 candidate rows,
one panel ahead of the words it updates.  The matrices here need many batches
(duplicated rows), find lower pivot columns in a later batch than higher ones
(anti-diagonal blocks), leave whole panels without a pivot, and cover every
word count with a full, a one-bit and a ragged last word.
"""

import numpy as np
import pytest

from hlf_inputs import low_rank_symmetric, random_symmetric
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu
from oracle import hlf_oracle as O
from test_gpu_factor import assert_record_matches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _anti(n):
    return np.eye(n, dtype=np.uint8)[::-1].copy()


def _repeated(n, distinct, seed):
    """Rows and columns repeat: row i is row i % distinct of a random core."""
    core = random_symmetric(distinct, seed, 0.5)
    i = np.arange(n) % distinct
    return core[np.ix_(i, i)].copy()


def _band(n):
    A = np.zeros((n, n), dtype=np.uint8)
    i = np.arange(n - 1)
    A[i, i + 1] = A[i + 1, i] = 1
    return A


def _late_rows(n, seed):
    """Only the last third of the rows touches the first third's columns."""
    A = np.zeros((n, n), dtype=np.uint8)
    k = n // 3
    B = (np.random.default_rng(seed).random((k, k)) < 0.5).astype(np.uint8)
    A[n - k :, :k] = B
    A[:k, n - k :] = B.T
    return A


def _gap(n, lo, hi, seed):
    """No row or column of [lo, hi): whole panels without a pivot."""
    A = random_symmetric(n, seed, 0.5)
    A[lo:hi, :] = 0
    A[:, lo:hi] = 0
    return A


def _cases():
    out = []
    for W in range(1, 17):
        for n in (64 * W, 64 * (W - 1) + 1, 64 * W - 29) if W < 7 else (64 * W - 29 * (W % 3),):
            out.append((f"random n={n}", random_symmetric(n, 77 + n, 0.5)))
    for n in (64, 65, 130, 192, 511, 900):
        out.append((f"anti n={n}", _anti(n)))
        out.append((f"band n={n}", _band(n)))
        out.append((f"late n={n}", _late_rows(n, n)))
    for n, d in ((128, 3), (300, 65), (640, 100), (900, 130)):
        out.append((f"repeated n={n} d={d}", _repeated(n, d, n + d)))
    for n, lo, hi in ((256, 0, 128), (256, 128, 256), (700, 60, 330), (1024, 64, 960)):
        out.append((f"gap n={n} {lo}..{hi}", _gap(n, lo, hi, n)))
    for n, k in ((320, 63), (320, 64), (320, 65), (800, 700)):
        out.append((f"low rank n={n} k={k}", low_rank_symmetric(n, k, n + k)))
    return out


@pytest.mark.parametrize("name,A", _cases(), ids=lambda x: x if isinstance(x, str) else "")
def test_panels_match_oracle(name, A):
    print(f"[panels] {name}", flush=True)
    F, st = gpu_factor(A, workgroup=True)
    assert st == hlf.HLF_OK
    assert_record_matches(F, O.factor(A), name)
