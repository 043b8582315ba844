"""First-stage expert tasks that work the routing out by themselves (up to 128 experts) or read it from the meta-tensor, while
the routing task is as late as it can be: every task delayed at random, with nothing requested ahead of an event, and with NaN in
whatever LDS nobody has written."""
import hashlib

import numpy as np
import pytest

import paper_2512_22219_amd as M
from synth import gen as G
from tests.gpu_util import GpuDecoder
from tests.test_compiler import own_routing

pytestmark = pytest.mark.gpu


def _digest(s, **opts):
    dec, h = GpuDecoder(s, 3, fusion=31, transitive_reduction=1, **opts), hashlib.sha256()
    for i in range(3):
        pos = np.array([(37 * b + 61) % (s.max_seq - 3) + i for b in range(s.batch)], np.int32)
        h.update(np.ascontiguousarray(dec.step(G.tokens(3 + i, s), pos)).tobytes())
    dec.close()
    return h.hexdigest()


@pytest.mark.parametrize("batch,experts,top_k", [(1, 128, 8), (4, 5, 5), (5, 129, 2), (16, 64, 16), (16, 65, 3)])
def test_same_bits_however_late(batch, experts, top_k):
    s = G.small_variant("C1", batch=batch, hidden=272, ffn=0, n_experts=experts, top_k=top_k, expert_ffn=64, vocab=1003)
    assert own_routing(s) == ({True} if experts <= 128 else {False})   # (or the comparisons are of one way with itself)
    assert own_routing(s, launch_mode=M.binding.LAUNCH_PER_OP) == {False}
    want = _digest(s)
    late = M.binding.DEBUG_JITTER | M.binding.DEBUG_POISON
    for opts in (dict(debug_flags=M.binding.DEBUG_JITTER), dict(debug_flags=late), dict(no_preload=1), dict(no_preload=1, debug_flags=late),
                 dict(launch_mode=M.binding.LAUNCH_PER_OP)):
        assert _digest(s, **opts) == want, opts
