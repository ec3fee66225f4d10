"""A rejected matrix has no rank: its result says 0 also where the device memory
of its record held another request's output before."""

import numpy as np
import pytest

from hlf_inputs import grid_instance
from paper_2103_00693_amd import hlf
from paper_2103_00693_amd.serve import Request, Server

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("N", [6, 9])
def test_rank_of_a_rejected_matrix(N):
    server = Server(slots=1, num_samples=65536, cache_entries=0, hbm_budget=64 << 20, host_budget=64 << 20)
    bad = grid_instance(N, seed=3)
    bad[0, N + 3] ^= 1
    for turn in range(3):
        print(f"[serve] rejected N={N} turn {turn}", flush=True)
        good = server.run([Request(rid=1, A=grid_instance(16, seed=turn), seed=turn)], realtime=False)[0]
        assert good.status == hlf.HLF_OK and np.any(good.data)
        res = server.run([Request(rid=2, A=bad, seed=5)], realtime=False)[0]
        assert (res.status, res.rank, res.kind) == (hlf.HLF_ENOTSYM, 0, "error") and res.data is None
