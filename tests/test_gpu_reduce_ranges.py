"""GPU parity of reduce mode at the edges of its tiles, for every word count:
ranges that begin and end inside a tile, in even and odd tiles, that hold one
tile or less, and disjoint ranges accumulated; and of the batched reduce at
ranks around the unit of its schedule.  Counts, hash and XOR-fold against the
oracle; integers, so equal or wrong.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import grid_instance, low_rank_symmetric
from oracle import c_oracle as C
from oracle import hlf_oracle as O
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _tile(W):
    """Indices per tile: 64 times the lane constants' unroll."""
    return 64 * (16 if W == 1 else 8 if W <= 3 else 4 if W <= 7 else 1)


def _check(F, Fo, begin, count, **kw):
    print(f"[reduce] n={Fo['n']} begin={begin} count={count}", flush=True)
    c, h, x = hlf.enumerate_reduce(F, begin, count, **kw)
    wc, wh, wx = C.reduce_range(Fo, begin, count)
    assert np.array_equal(hlf.as_uint64(c), wc)
    assert int(hlf.as_uint64(h)[0]) == int(wh)
    assert np.array_equal(hlf.as_uint64(x), wx)


@pytest.mark.parametrize("W", range(1, 17))
def test_ranges(W):
    n = 64 * W - (0 if W % 3 == 0 else 5 * W % 61)
    A = low_rank_symmetric(n, 15, W)
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    t, top = _tile(W), 1 << Fo["rank"]
    ranges = [(0, 1), (1, 1), (0, t), (t, t), (t - 1, 2), (3, t - 7), (t + 3, t - 7), (2 * t - 1, 1), (t + 5, 2 * t), (1, 3 * t),
              (3 * t + 1, 2 * t + 1), (0, top), (1, top - 2), (top - 1, 1), (top - t - 1, t + 1)]
    for begin, count in ranges:
        if begin + count <= top:
            _check(F, Fo, begin, count)
    assert int(F.status.item()) == hlf.HLF_OK


@pytest.mark.parametrize("n,k", [(25, 20), (70, 17), (200, 16), (577, 14), (1024, 13)])
def test_accumulate_disjoint_ranges(n, k):
    A = grid_instance(5, seed=3) if n == 25 else low_rank_symmetric(n, k, 5)
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    top = 1 << min(Fo["rank"], 20)
    cuts = [0, 1, 777, 778, top // 3, top // 2 + 13, top]
    out = None
    for lo, hi in zip(cuts, cuts[1:]):
        if out is None:
            out = hlf.enumerate_reduce(F, lo, hi - lo)
        else:
            hlf.enumerate_reduce(F, lo, hi - lo, accumulate=True, counts=out[0], hash_out=out[1], xorfold=out[2])
    wc, wh, wx = C.reduce_range(Fo, 0, top)
    assert np.array_equal(hlf.as_uint64(out[0]), wc)
    assert int(hlf.as_uint64(out[1])[0]) == int(wh)
    assert np.array_equal(hlf.as_uint64(out[2]), wx)


def test_high_indices():
    """Tiles whose index has its high bits set (r > 50)."""
    A = grid_instance(8, 0.5, 0)
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    r = Fo["rank"]
    assert 50 < r <= 62
    for begin in ((1 << (r - 1)) - 777, (0x5555555555555555 & ((1 << r) - 1)) - 5000, (1 << r) - 3001):
        _check(F, Fo, begin, 3001)


def test_empty_range_zeroes_or_keeps():
    A = grid_instance(4, seed=1)
    F, _ = gpu_factor(A)
    c = torch.full((16,), 7, dtype=torch.int64, device="cuda")
    h, x = torch.full((1,), 7, dtype=torch.int64, device="cuda"), torch.full((1,), 7, dtype=torch.int64, device="cuda")
    hlf.enumerate_reduce(F, 5, 0, accumulate=True, counts=c, hash_out=h, xorfold=x)
    assert (c == 7).all() and int(h) == 7 and int(x) == 7
    hlf.enumerate_reduce(F, 5, 0, counts=c, hash_out=h, xorfold=x)
    assert (c == 0).all() and int(h) == 0 and int(x) == 0


@pytest.mark.parametrize("max_rank", [0, 9, 16, 17, 18, 20])
@pytest.mark.parametrize("params", [None, (10, 1), (17, 16), (22, 4)])
def test_batch_units(max_rank, params):
    """Instances of rank 0 to 20 (and larger ones, which are skipped) in units
    of 2^10 to 2^22; a matrix that is not symmetric among them."""
    mats = [np.zeros((5, 5), dtype=np.uint8)]
    mats += [low_rank_symmetric(n, k, 7 * n + k) for n in (40, 64, 65, 130, 192) for k in (1, 2, 9, 16, 17, 18, 20)]
    mats += [grid_instance(N, seed=N) for N in (3, 4, 6)]
    bad = grid_instance(4, seed=2)
    bad[0, 5] ^= 1
    mats.append(bad)
    Fo = [O.factor(A) for A in mats[:-1]]
    B = hlf.Batch([A.shape[0] for A in mats])
    print(f"[reduce] batch max_rank={max_rank} params={params}", flush=True)
    B.reduce(B.dense_input(mats), max_rank, None if params is None else hlf.BatchParams(*params))
    counts, hashes = B.reduce_results()
    assert list(B.statuses()) == [hlf.HLF_OK] * len(Fo) + [hlf.HLF_ENOTSYM]
    for i, f in enumerate(Fo):
        if f["rank"] <= max_rank:
            wc, wh, _ = C.reduce_range(f, 0, 1 << f["rank"])
            assert np.array_equal(counts[i], wc) and hashes[i] == int(wh), i
        else:
            assert not counts[i].any() and hashes[i] == 0, i
    assert not counts[-1].any() and hashes[-1] == 0
