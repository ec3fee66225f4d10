"""Records published between workgroups inside one launch, many launches over:
the arrays hold other values before each, so a record that is read before its
writer's stores have arrived gives another hash or other solutions.  Results
are compared on the device with those of separate launches.
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


def _hashes(mats):
    out = []
    for A in mats:
        F, st = gpu_factor(A)
        assert st == hlf.HLF_OK
        out.append(hlf.enumerate_reduce(F, 0, 1 << int(F.rank.item()))[1])
    return torch.cat(out)


@pytest.mark.parametrize("count,waves,chunk,repeats", [(40, 8, 20, 2000), (500, 8, 12, 2000), (500, 1, 20, 500), (3000, 12, 17, 300)])
def test_reduce_reads_published_records(count, waves, chunk, repeats):
    pool = [grid_instance(1 + i % 3, (0.5, 1.0)[i % 2], i) for i in range(60)]
    for i in range(20):  # two and three words
        A = np.zeros((70 + 6 * i, 70 + 6 * i), dtype=np.uint8)
        A[-8:, -8:] = random_symmetric(8, i, 0.5)
        pool.append(A)
    at = [(i * 37) % len(pool) for i in range(count)]
    ns = np.array([pool[k].shape[0] for k in at], dtype=np.int64)
    Ws = (ns + 63) // 64
    A_dev = torch.from_numpy(np.concatenate([pool[k].reshape(-1) for k in at])).cuda()
    n_dev = torch.from_numpy(ns.astype(np.int32)).cuda()
    want = _hashes(pool)[torch.tensor(at, device="cuda")]
    i32, i64 = torch.int32, torch.int64
    sizes = {"status": (count, i32), "rank": (count, i32), "pivots": (ns.sum(), i32), "basis": ((ns * Ws).sum(), i64),
             "shift": (Ws.sum(), i64), "counts": (ns.sum(), i64), "hash": (count, i64)}
    out = {k: torch.empty(int(m), dtype=dt, device="cuda") for k, (m, dt) in sizes.items()}
    out["kernel"] = None
    wrong = torch.zeros((), dtype=i64, device="cuda")
    params = hlf.BatchParams(chunk, waves)
    for _ in range(repeats):
        for k in ("rank", "basis", "shift", "hash"):
            out[k].fill_(7)  # a rank of 7 and rows of 7: in range, and another hash
        hlf.batch_reduce_noalloc(n_dev, int(ns.max()), A_dev, 9, out, params)
        wrong += (out["hash"] != want).sum()
    print(f"[publish] {count} instances, {repeats} launches, wrong hashes {int(wrong.item())}", flush=True)
    assert int(wrong.item()) == 0


def test_solve_reads_published_records():
    """Two sets of matrices in turn through one batch's records."""
    sets = [[grid_instance(4, 1.0, 2 * s + t) for s in range(8)] for t in range(2)]
    B = hlf.Batch([16] * 8)
    inputs = [B.dense_input(m) for m in sets]
    # the first solutions of each, as many as both sets have
    ranks = [[int(gpu_factor(A)[0].rank.item()) for A in m] for m in sets]
    counts = [1 << min(a, b) for a, b in zip(*ranks)]
    wants = []
    for m in sets:
        wants.append([hlf.enumerate_solutions(gpu_factor(A)[0], 0, c, 32) for A, c in zip(m, counts)])
    outs = [torch.empty(c, dtype=torch.int32, device="cuda") for c in counts]
    wrong = torch.zeros((), dtype=torch.int64, device="cuda")
    for k in range(1000):
        B.solve(inputs[k & 1], list(range(8)), [0] * 8, counts, outs, 32)
        for o, w in zip(outs, wants[k & 1]):
            wrong += (o != w).sum()
    assert int(wrong.item()) == 0
