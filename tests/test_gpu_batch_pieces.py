"""Batches of every weight: the length of the reduce pieces and the size of the
grid go with the instance count and max_rank, and short pieces are taken in
turn instead of drawn.  Counts and hash of each instance against the
single-instance reduce of its own record.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import grid_instance, random_symmetric
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _mats(count):
    """Grids of sides 1 to 9 in turn (one, two words), every fifth a sparse graph of three."""
    out = []
    for i in range(count):
        if i % 5 == 4:
            A = np.zeros((150, 150), dtype=np.uint8)
            k = 3 + i % 14
            A[140 - k : 140, 140 - k : 140] = random_symmetric(k, i, 0.5)
            out.append(A)
        else:
            out.append(grid_instance(1 + i % 9 if i % 3 else 4, (0.3, 0.5, 1.0)[i % 3], i))
    return out


_single = {}


def _reference(i, A, max_rank):
    if i not in _single:
        F, st = gpu_factor(A)
        assert st == hlf.HLF_OK
        _single[i] = (F, int(F.rank.item()), {})
    F, r, done = _single[i]
    if r > max_rank:
        return r, np.zeros(A.shape[0], dtype=np.uint64), 0
    if "c" not in done:
        c, h, _ = hlf.enumerate_reduce(F, 0, 1 << r)
        done["c"], done["h"] = c.cpu().numpy().view(np.uint64), int(h.item()) & ((1 << 64) - 1)
    return r, done["c"], done["h"]


# (instances, max_rank, chunk_log2, waves per CU): the shortest pieces, the bounds
# between short and drawn ones, fewer waves than tasks and more, caller's chunks
CASES = [(1, 0, 20, 8), (1, 16, 20, 8), (1, 24, 20, 8), (3, 12, 20, 8), (40, 13, 20, 8), (40, 16, 20, 8),
         (40, 20, 10, 8), (40, 24, 20, 1), (300, 14, 20, 1), (300, 18, 16, 2), (300, 20, 20, 8), (300, 21, 11, 16),
         (300, 24, 17, 8)]


@pytest.mark.parametrize("count,max_rank,chunk,waves", CASES)
def test_against_single_reduce(count, max_rank, chunk, waves):
    print(f"[pieces] {count} instances, max_rank {max_rank}, chunk 2^{chunk}, {waves} waves", flush=True)
    mats = _mats(count)
    ns = np.array([A.shape[0] for A in mats], dtype=np.int64)
    Ws = (ns + 63) // 64
    A_dev = torch.from_numpy(np.concatenate([A.reshape(-1) for A in mats])).cuda()
    n_dev = torch.from_numpy(ns.astype(np.int32)).cuda()

    def fives(k, dt):
        return torch.full((int(k),), 5, dtype=dt, device="cuda")

    i32, i64 = torch.int32, torch.int64
    out = {"status": fives(count, i32), "rank": fives(count, i32), "pivots": fives(ns.sum(), i32),
           "basis": fives((ns * Ws).sum(), i64), "shift": fives(Ws.sum(), i64), "kernel": None,
           "counts": fives(ns.sum(), i64), "hash": fives(count, i64)}
    for _ in range(2):
        hlf.batch_reduce_noalloc(n_dev, int(ns.max()), A_dev, max_rank, out, hlf.BatchParams(chunk, waves))
    B = hlf.Batch([int(n) for n in ns])
    B.reduce(B.dense_input(mats), max_rank, hlf.BatchParams(chunk, waves))
    bc, bh = B.reduce_results()
    counts = out["counts"].cpu().numpy().view(np.uint64)
    hashes = out["hash"].cpu().numpy().view(np.uint64)
    at = 0
    for i, A in enumerate(mats):
        r, c, h = _reference(i, A, max_rank)
        n = A.shape[0]
        assert int(out["rank"][i]) == r, i
        assert np.array_equal(counts[at : at + n], c) and int(hashes[i]) == h, (i, r)
        assert np.array_equal(bc[i], c) and bh[i] == h, (i, r)
        at += n
