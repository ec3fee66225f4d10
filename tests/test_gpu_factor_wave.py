"""The one-wavefront stage 1 (batches, n <= 192) at its edges, bit for bit
against the oracle: every n up to 20 and around each word and half-word, the
matrices one after the other in memory and so at any address, with full, small
and no rank, and a bad byte or an asymmetric pair anywhere in the last load.
"""

import numpy as np
import pytest

from hlf_inputs import grid_instance, low_rank_symmetric, random_symmetric
from paper_2103_00693_amd import hlf

from gpu_util import require_gpu
from oracle import hlf_oracle as O

pytestmark = pytest.mark.gpu

EDGES = sorted({m + d for m in (32, 64, 96, 128, 160) for d in (-1, 0, 1)} | {81, 100, 121, 144, 177, 191, 192})


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _mats(kind):
    out = []
    for n in list(range(1, 21)) + EDGES:
        if kind == "dense":
            out.append(random_symmetric(n, 31 * n, 0.5))
        elif kind == "sparse":
            out.append(random_symmetric(n, 37 * n, 2.0 / n))
        elif kind == "zero":
            out.append(np.zeros((n, n), dtype=np.uint8))
        elif kind == "anti":
            out.append(np.eye(n, dtype=np.uint8)[::-1].copy())
        elif kind == "low rank":
            out.append(low_rank_symmetric(n, max(1, n // 5), n))
        else:
            N = max(1, int(round(n**0.5)))
            out.append(grid_instance(N, 0.3, n))
    return out


@pytest.mark.parametrize("kind", ["dense", "sparse", "zero", "anti", "low rank", "grid"])
def test_records(kind):
    mats = _mats(kind)
    print(f"[wave] {kind}: {len(mats)} instances", flush=True)
    B = hlf.Batch([m.shape[0] for m in mats])
    B.factor_dense(B.dense_input(mats))
    for A, got in zip(mats, B.records()):
        n, ref = A.shape[0], O.factor(A)
        r = ref["rank"]
        assert got["status"] == hlf.HLF_OK and got["rank"] == r, n
        assert list(got["pivots"][:r]) == ref["pivots"] and all(p == -1 for p in got["pivots"][r:]), n
        assert got["basis"] == ref["basis"] and got["shift"] == ref["shift"], n
        assert got["kernel"] == ref["kernel"], n


def test_bad_entries_in_the_last_load():
    mats, want = [], []
    for n in list(range(1, 21)) + EDGES:
        for fault in ("none", "last byte", "first byte", "pair", "corner"):
            A = random_symmetric(n, n, 0.5)
            if fault == "last byte":
                A[n - 1, n - 1] = 2
            elif fault == "first byte":
                A[0, 0] = 129
            elif fault == "pair" and n > 1:
                A[n - 1, n - 2] ^= 1
            elif fault == "corner" and n > 1:
                A[0, n - 1] ^= 1
            mats.append(A)
            want.append(hlf.HLF_OK if fault == "none" or (n == 1 and fault in ("pair", "corner")) else hlf.HLF_ENOTSYM)
    B = hlf.Batch([m.shape[0] for m in mats])
    B.factor_dense(B.dense_input(mats))
    assert list(B.statuses()) == want
