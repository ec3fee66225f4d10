"""GPU parity of the kernels that write one 16-byte store per thread: ranges
that begin and end anywhere inside a store, a wave's run or a 4 KiB tile, at
any address, in both orders and all word sizes, alone and as tasks of a batch,
and the circuit over the same edges.  Words around the output must stay as
they were.  Integers: results are equal or wrong.
"""

import numpy as np
import pytest
import torch

from hlf_inputs import grid_instance
from oracle import c_oracle as C
from oracle import hlf_oracle as O
from paper_2103_00693_amd import hlf

from gpu_util import device_matrix, gpu_factor, narrow_to_u64, require_gpu

pytestmark = pytest.mark.gpu

DTYPES = {16: torch.int16, 32: torch.int32, 64: torch.int64}
GUARD = 40  # words checked before and after the output


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _out(count, bits, shift):
    """A guarded output of `count` words, `shift` words past a 16-byte boundary."""
    buf = torch.full((GUARD + shift + count + GUARD,), 0x5A, dtype=DTYPES[bits], device="cuda")
    lead = (-buf.data_ptr() // (bits // 8)) % (16 // (bits // 8))
    a = GUARD - GUARD % (16 // (bits // 8)) + lead + shift if lead else GUARD + shift
    assert a + count <= buf.numel()
    return buf, a


def _check(buf, a, count, want):
    torch.cuda.synchronize()
    got = narrow_to_u64(buf)
    mask = (1 << (8 * buf.element_size())) - 1
    assert np.array_equal(got[a:a + count], want & np.uint64(mask))
    assert (got[:a] == 0x5A).all() and (got[a + count:] == 0x5A).all()


def _ranges(bits, r):
    V = 16 // (bits // 8)
    tile, run, top = 256 * V, 64 * V, 1 << r
    rng = [(0, 1), (1, 1), (V - 1, 2), (1, run), (run - 1, 2), (3, tile - 3), (0, tile), (0, tile + 1), (tile - 1, 2),
           (5, 3 * tile), (2 * tile, 2 * tile), (7 * tile + 1, 9 * tile + V - 1), (top - 1, 1), (top - tile - 3, tile + 3)]
    return [(b, c) for b, c in rng if b >= 0 and b + c <= top]


@pytest.mark.parametrize("order", ["gray", "counter"])
@pytest.mark.parametrize("bits", [16, 32, 64])
@pytest.mark.parametrize("N,seed", [(1, 0), (1, 1), (2, 3), (3, 1), (4, 0), (5, 2), (6, 4), (8, 0)])
def test_ranges_and_addresses(N, seed, bits, order):
    if N * N > bits:
        pytest.skip("word too narrow for this grid")
    A = grid_instance(N, 0.5 if N == 8 else 1.0, seed)  # a rank of at most 62
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    r = min(Fo["rank"], 40)
    ref = C.enumerate_range if order == "gray" else C.enumerate_counter_range
    for begin, count in _ranges(bits, r):
        want = ref(Fo, begin, count)[:, 0]
        for shift in (0, 1, 3):
            print(f"[vec] N={N} bits={bits} {order} begin={begin} count={count} shift={shift}", flush=True)
            buf, a = _out(count, bits, shift)
            hlf.enumerate_solutions(F, begin, count, bits, out=buf[a:], order=order)
            _check(buf, a, count, want)
    assert int(F.status.item()) == hlf.HLF_OK


def test_high_index_bits():
    """Runs whose first index has its high bits set (n = 64)."""
    A = grid_instance(8, 0.5, 0)
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    r = Fo["rank"]
    assert 50 < r <= 62
    for begin in ((1 << (r - 1)) - 777, (0x5555555555555555 & ((1 << r) - 1)) - 5000, (1 << r) - 3001):
        for order, ref in (("gray", C.enumerate_range), ("counter", C.enumerate_counter_range)):
            buf, a = _out(3001, 64, 1)
            hlf.enumerate_solutions(F, begin, 3001, 64, out=buf[a:], order=order)
            _check(buf, a, 3001, ref(Fo, begin, 3001)[:, 0])


@pytest.mark.parametrize("begin,count", [(0, (1 << 9) + 1), (1 << 9, 1), ((1 << 64) - 4, 8), (1 << 63, 1 << 62)])
def test_range_errors_write_nothing(begin, count):
    A = grid_instance(3, b="1" * 9)
    F, _ = gpu_factor(A)
    assert int(F.rank.item()) <= 9
    buf, a = _out(600, 16, 0)
    hlf.enumerate_solutions(F, begin, count, 16, out=buf[a:])
    _check(buf, a, 0, np.zeros(0, dtype=np.uint64))
    assert int(F.status.item()) == hlf.HLF_ERANGE


@pytest.mark.parametrize("num", [1, 2, 15, 16, 17, 35])
@pytest.mark.parametrize("bits", [32, 64])
def test_batch_tasks(num, bits):
    """Mixed instances as tasks of one launch (16 at most): repeated and
    skipped instances, empty ranges, odd begins and addresses."""
    rng = np.random.default_rng(num * 100 + bits)
    mats = [grid_instance(int(N), seed=int(s)) for N, s in zip(rng.integers(1, 6, 12), rng.integers(0, 1 << 30, 12))]
    Fo = [O.factor(A) for A in mats]
    B = hlf.Batch([A.shape[0] for A in mats])
    B.factor_dense(B.dense_input(mats))
    inst, begins, counts, outs, bufs = [], [], [], [], []
    for k in range(num):
        i = int(rng.integers(0, len(mats)))
        top = 1 << Fo[i]["rank"]
        c = int(min(top, rng.choice([0, 1, 5, 900, 5000, 70000])))
        b = int(rng.integers(0, top - c + 1))
        buf, a = _out(c, bits, int(rng.integers(0, 4)))
        inst.append(i), begins.append(b), counts.append(c), outs.append(buf[a:]), bufs.append((buf, a))
    print(f"[vec] batch num={num} bits={bits} {list(zip(inst, begins, counts))}", flush=True)
    B.enumerate(inst, begins, counts, outs, bits)
    for i, b, c, (buf, a) in zip(inst, begins, counts, bufs):
        _check(buf, a, c, C.enumerate_range(Fo[i], b, c)[:, 0] if c else np.zeros(0, dtype=np.uint64))


def test_batch_bad_task_leaves_the_others():
    mats = [grid_instance(4, seed=s) for s in range(3)]
    Fo = [O.factor(A) for A in mats]
    B = hlf.Batch([16] * 3)
    B.factor_dense(B.dense_input(mats))
    counts = [1 << Fo[0]["rank"], (1 << Fo[1]["rank"]) + 1, 1 << Fo[2]["rank"]]
    bufs = [_out(c, 32, 1) for c in counts]
    B.enumerate([0, 1, 2], [0] * 3, counts, [buf[a:] for buf, a in bufs], 32)
    for k in (0, 2):
        _check(*bufs[k], counts[k], C.enumerate_range(Fo[k], 0, counts[k])[:, 0])
    _check(*bufs[1], 0, np.zeros(0, dtype=np.uint64))
    assert list(B.statuses()) == [hlf.HLF_OK, hlf.HLF_ERANGE, hlf.HLF_OK]


@pytest.mark.parametrize("bits", [16, 32, 64])
@pytest.mark.parametrize("N,p,seed", [(1, 1.0, 1), (2, 1.0, 3), (3, 1.0, 1), (4, 1.0, 0), (4, 0.5, 2), (5, 0.5, 3), (7, 0.5, 4),
                                      (8, 0.5, 0)])
def test_circuit_ranges(N, p, seed, bits):
    if N * N > bits:
        pytest.skip("word too narrow for this grid")
    A = grid_instance(N, p, seed)
    Fo = O.factor(A)
    rows, _ = hlf.pack_dense(device_matrix(A))
    F = hlf.factor(rows, N * N)
    V = 16 // (bits // 8)
    for begin, count in _ranges(bits, min(Fo["rank"], 40)):
        begin -= begin % V
        print(f"[vec] circuit N={N} bits={bits} begin={begin} count={count}", flush=True)
        buf, a = _out(count, bits, 0)
        hlf.enumerate_circuit(F, rows, N, begin, count, bits, out=buf[a:])
        _check(buf, a, count, C.enumerate_counter_range(Fo, begin, count)[:, 0])
    assert int(F.status.item()) == hlf.HLF_OK


@pytest.mark.parametrize("N,u,v", [(3, 2, 3), (4, 0, 5), (5, 4, 5), (8, 0, 63), (8, 7, 8)])
def test_circuit_refuses_entries_off_the_grid(N, u, v):
    """An entry between vertices that are no grid neighbours (among them the
    end of one row and the start of the next)."""
    A = grid_instance(N, 0.5, 1)
    A[u, v] = A[v, u] = 1
    rows, _ = hlf.pack_dense(device_matrix(A))
    F = hlf.factor(rows, N * N)
    bits = 64
    buf, a = _out(8, bits, 0)
    hlf.enumerate_circuit(F, rows, N, 0, 8, bits, out=buf[a:])
    _check(buf, a, 0, np.zeros(0, dtype=np.uint64))
    assert int(F.status.item()) == hlf.HLF_EINVAL
