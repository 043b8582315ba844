"""Logits to the last bit, as digests.  Every order of additions and every rounding of a step is in them: where the compiler
contracts a product and a sum, how lanes are added, which chunk of a row comes first.  None of that may move by accident,
since single appended bf16 rows then round the other way and whole outputs follow.  (An order that is changed on
purpose replaces the digests of its shapes, once its error against 64 bits has been measured on both sides.)"""
import hashlib

import numpy as np
import pytest

from synth import gen as G
from tests.gpu_util import GpuDecoder

pytestmark = pytest.mark.gpu

# query/key norm: both head sizes, every number of query heads per KV head, every batch class
QK = [
    (dict(batch=1), "b7a891c06893f22a"),
    (dict(batch=2, head_dim=128, n_q_heads=8, n_kv_heads=2), "72ef15ebe6255e24"),
    (dict(batch=4, n_q_heads=4, n_kv_heads=4), "13ca3ae8c2434767"),
    (dict(batch=8, n_q_heads=16, n_kv_heads=2), "c8ff342fd2eadd28"),
    (dict(batch=16, head_dim=128, n_q_heads=4, n_kv_heads=4), "542f55c5d32deb73"),
    (dict(batch=3, head_dim=128, n_q_heads=16, n_kv_heads=2, ffn=0, n_experts=16, top_k=4, expert_ffn=64), "c8ac03d31c182d51"),
]
# without: rows of two segments, and of 2048 inputs at batch 2 (20 chunks a sequence); mixture of experts
PLAIN = [
    (dict(batch=1, hidden=4104, vocab=1003), "12addd4eaff60de6"),
    (dict(batch=2, hidden=2048, n_q_heads=16, n_kv_heads=2, max_seq=2624), "42d12e09459fd6f2"),
    (dict(batch=1, ffn=0, n_experts=16, top_k=4, expert_ffn=64), "a9b57e659cf7bfff"),
]


def digest(kw):
    s = G.small_variant("C1", **kw)
    dec, h = GpuDecoder(s, 3, fusion=31, transitive_reduction=1, n_workers=256), hashlib.sha256()
    for i in range(2):
        pos = np.array([(37 * b + 61) % (s.max_seq - 2) + i for b in range(s.batch)], np.int32)
        h.update(np.ascontiguousarray(dec.step(G.tokens(3 + i, s), pos)).tobytes())
    dec.close()
    return h.hexdigest()[:16]


@pytest.mark.parametrize("kw,want", [(dict(qk_norm=True, **kw), want) for kw, want in QK] + PLAIN)
def test_logits_to_the_bit(kw, want):
    assert digest(kw) == want
