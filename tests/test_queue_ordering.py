"""Memory orders of the batch reduce's work queue, read from its source (the
hardware may keep an order that the source does not ask for, so no run shows a
missing one).  A wave may leave when no chunk is left for it: it has to decide
that on one claim word, whose own slots say that no claim is still to come, and
not on a second counter that nothing orders behind the claims.  A published
entry has to come after a release of the record behind it, and its reader to
acquire it.
"""

import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2103_00693_amd", "csrc", "batch.hip")


def _kernel():
    src = re.sub(r"//[^\n]*", "", open(SRC).read())
    body = src[src.index("void batch_reduce_kernel("):]
    return re.sub(r"\s+", " ", body[: body.index("struct hlf_batch_s")])


def test_waves_leave_on_the_claim_word_alone():
    k = _kernel()
    # one read of the claims per look, and the test to leave is on its slots
    assert k.count("relaxed_load(&q->claim)") == 1
    leave = [m for m in re.findall(r"if \(([^;{}]*?)\) break;", k) if "cl >> kClaimShift" in m]
    assert leave == ["(unsigned int)(cl >> kClaimShift) + skipped >= (unsigned int)b.count"]
    # a task claims or is counted, never both
    claims = k.index("atomicAdd(&q->claim")
    assert k.count("atomicAdd(&q->claim") == 1 and k.count("fetch_add(&q->fskip") == 1
    assert re.search(r"\} else if \(lane == 0\) \{ __hip_atomic_fetch_add\(&q->fskip", k[claims:])


def test_entries_release_and_acquire_their_records():
    k = _kernel()
    assert len(re.findall(r"__hip_atomic_store\(&slots\[", k)) == 1
    written, stored = k.index("b.hash[f] = 0"), k.index("__hip_atomic_store(&slots[")
    assert "release_to_device();" in k[written:stored]
    found = k.index("find_slot(slots,")
    assert '__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent")' in k[found : k.index("b.rank[inst]")]
