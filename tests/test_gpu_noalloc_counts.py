"""hlf_batch_reduce_noalloc above 1024 instances, where a thread of its layout
launch adds up several sizes: records and results against hlf_batch_reduce of
the same instances, at counts that leave the last threads short or empty, and
with entries of n_dev that are no size (they take no space and are refused).
"""

import numpy as np
import pytest
import torch

from hlf_inputs import grid_instance
from paper_2103_00693_amd import hlf

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

MAX_RANK = 14


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _mat(i):
    if i % 97 == 96:  # two and three words, a small rank
        A = np.zeros((70 + i % 110,) * 2, dtype=np.uint8)
        A[-9:, -9:] = grid_instance(3, seed=i)
        return A
    return grid_instance(1 + i % 4, (0.3, 0.5, 1.0)[i % 3], i)


@pytest.mark.parametrize("count,refused", [(1024, 0), (1025, 0), (1025, 3), (2047, 5), (5000, 0), (16384, 7)])
def test_against_batch_reduce(count, refused):
    print(f"[noalloc] {count} instances, {refused} refused", flush=True)
    pool = [_mat(i) for i in range(388)]
    mats = [pool[(i * 131) % 388] for i in range(count)]
    ns = np.array([A.shape[0] for A in mats], dtype=np.int64)
    Ws = (ns + 63) // 64
    max_n = int(ns.max())
    # refused entries stand between the others: n_dev has count of them in all
    places = set(np.linspace(1, count - 1, refused).astype(int)) if refused else set()
    keep = [i for i in range(count) if i not in places]
    n_all = ns.astype(np.int32)
    n_all[sorted(places)] = [(0, -5, max_n + 1, 1 << 30)[k % 4] for k in range(len(places))]
    A_dev = torch.from_numpy(np.concatenate([mats[i].reshape(-1) for i in keep])).cuda()
    n_dev = torch.from_numpy(n_all).cuda()

    def fives(k, dt):
        return torch.full((int(k),), 5, dtype=dt, device="cuda")

    i32, i64 = torch.int32, torch.int64
    kn, kW = ns[keep], Ws[keep]
    out = {"status": fives(count, i32), "rank": fives(count, i32), "pivots": fives(kn.sum(), i32),
           "basis": fives((kn * kW).sum(), i64), "shift": fives(kW.sum(), i64), "kernel": fives((kn * kW).sum(), i64),
           "counts": fives(kn.sum(), i64), "hash": fives(count, i64)}
    hlf.batch_reduce_noalloc(n_dev, max_n, A_dev, MAX_RANK, out)
    B = hlf.Batch([int(n) for n in kn])
    B.reduce(A_dev, MAX_RANK)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    status, rank = B.statuses(), B.ranks()
    assert np.array_equal(got["status"][keep], status) and (status == hlf.HLF_OK).all()
    assert np.array_equal(got["rank"][keep], rank)
    for i in places:
        assert got["status"][i] == hlf.HLF_EINVAL and got["rank"][i] == 0
    assert np.array_equal(got["pivots"], B._read("pivots", 4 * int(kn.sum()), np.int32))
    assert np.array_equal(got["shift"], B._read("shift", 8 * int(kW.sum()), np.int64))
    assert np.array_equal(got["counts"], B._read("counts", 8 * int(kn.sum()), np.int64))
    assert np.array_equal(got["hash"][keep], B._read("hash", 8 * len(keep), np.int64))
    basis, kernel = (B._read(k, 8 * int((kn * kW).sum()), np.int64) for k in ("basis", "kernel"))
    at = 0  # rows past the rank, and past n - r, are not written
    for n, W, r in zip(kn, kW, rank):
        assert np.array_equal(got["basis"][at : at + r * W], basis[at : at + r * W])
        assert np.array_equal(got["kernel"][at : at + (n - r) * W], kernel[at : at + (n - r) * W])
        at += n * W
