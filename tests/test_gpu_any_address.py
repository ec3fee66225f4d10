"""hlf_enumerate and hlf_batch_enumerate into outputs at any byte address
(tensors of whole words cannot be placed there, so these go through the C ABI):
one word per solution in every size, two to sixteen words, both orders, ranges
inside one tile and over several, the bytes around the output untouched.
Integers: results are equal or wrong.
"""

import ctypes

import numpy as np
import pytest
import torch

from hlf_inputs import grid_instance, low_rank_symmetric
from oracle import c_oracle as C
from oracle import hlf_oracle as O
from paper_2103_00693_amd import hlf

from gpu_util import gpu_factor, require_gpu

pytestmark = pytest.mark.gpu

GUARD = 64  # bytes checked before and after the output


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _buffer(nbytes, offset):
    buf = torch.full((GUARD + 16 + nbytes + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    assert buf.data_ptr() % 16 == 0
    return buf, GUARD + offset


def _check(buf, at, want):
    got = buf.cpu().numpy()
    raw = np.ascontiguousarray(want).view(np.uint8).reshape(-1)
    assert np.array_equal(got[at : at + raw.size], raw)
    assert (got[:at] == 0xA5).all() and (got[at + raw.size :] == 0xA5).all()


def _narrow(z, bits):
    return z[:, 0].astype({16: np.uint16, 32: np.uint32, 64: np.uint64}[bits])


@pytest.mark.parametrize("offset", [1, 2, 3, 4, 6, 7, 9, 15])
@pytest.mark.parametrize("bits,N", [(16, 4), (32, 5), (64, 6)])
def test_one_word(bits, N, offset):
    A = grid_instance(N, seed=1)
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    V = 128 // bits
    for flags, ref in ((0, C.enumerate_range), (hlf.HLF_ORDER_COUNTER, C.enumerate_counter_range)):
        for begin, count in ((0, 1), (1, V + 1), (V, 256 * V), (3, 2 * 256 * V + 5)):
            want = _narrow(ref(Fo, begin, count), bits)
            buf, at = _buffer(want.nbytes, offset)
            print(f"[address] {bits} bits, offset {offset}, begin {begin}, count {count}, flags {flags}", flush=True)
            st = hlf.lib().hlf_enumerate_ex(F.c, begin, count, bits, flags, buf.data_ptr() + at, hlf._stream())
            assert st == hlf.HLF_OK
            _check(buf, at, want)
    assert int(F.status.item()) == hlf.HLF_OK


@pytest.mark.parametrize("offset", [1, 2, 4, 8, 11])
@pytest.mark.parametrize("n", [70, 128, 192, 256, 300, 510, 1024])
def test_several_words(n, offset):
    A = low_rank_symmetric(n, 14, n)
    Fo = O.factor(A)
    F, _ = gpu_factor(A)
    W = hlf.words_for(n)
    top = 1 << Fo["rank"]
    assert top >= 2048
    for flags, ref in ((0, C.enumerate_range), (hlf.HLF_ORDER_COUNTER, C.enumerate_counter_range)):
        for begin, count in ((0, 1), (5, 100), (0, 512), (77, 1301), (top - 3, 3)):
            want = ref(Fo, begin, count)
            buf, at = _buffer(want.nbytes, offset)
            print(f"[address] {W} words, offset {offset}, begin {begin}, count {count}, flags {flags}", flush=True)
            st = hlf.lib().hlf_enumerate_ex(F.c, begin, count, 64 * W, flags, buf.data_ptr() + at, hlf._stream())
            assert st == hlf.HLF_OK
            _check(buf, at, want)
    assert int(F.status.item()) == hlf.HLF_OK


@pytest.mark.parametrize("bits", [16, 32, 64])
def test_batch_tasks(bits):
    mats = [grid_instance(4, seed=s) for s in range(5)]
    Fo = [O.factor(A) for A in mats]
    B = hlf.Batch([16] * 5)
    B.factor_dense(B.dense_input(mats))
    begins, offsets = [0, 1, 2, 7, 100], [1, 2, 5, 8, 13]
    counts = [(1 << f["rank"]) - b for f, b in zip(Fo, begins)]
    wants = [_narrow(C.enumerate_range(f, b, c), bits) for f, b, c in zip(Fo, begins, counts)]
    bufs = [_buffer(w.nbytes, o) for w, o in zip(wants, offsets)]
    i32, u64, vp = ctypes.c_int32, ctypes.c_uint64, ctypes.c_void_p
    st = hlf._batch_lib().hlf_batch_enumerate(
        B._h, 5, (i32 * 5)(*range(5)), (u64 * 5)(*begins), (u64 * 5)(*counts),
        (vp * 5)(*[buf.data_ptr() + at for buf, at in bufs]), bits, hlf._stream())
    assert st == hlf.HLF_OK
    for (buf, at), want in zip(bufs, wants):
        _check(buf, at, want)
    assert (B.statuses() == hlf.HLF_OK).all()
