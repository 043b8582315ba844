"""The kernel sets whose kernels spill vector registers beside scalar ones (large tasks, and two rows), above all their hybrid
walks: the plain, the hybrid and the per-operator launch run the same task bodies in kernels that spill differently, so
logits have to be equal to the last bit, with and without random delays."""
import numpy as np
import pytest

import paper_2512_22219_amd as M
from synth import gen as G
from synth.device import DeviceModel
from tests.gpu_util import GpuDecoder

pytestmark = pytest.mark.gpu

SETS = [   # batch class of the set, shape, workers
    (9, dict(hidden=1024, ffn=4096, n_q_heads=8, n_kv_heads=2, vocab=2003), 5),      # large tasks: three weight buffers
    (9, dict(hidden=4104, ffn=4104, n_layers=3, vocab=1003, qk_norm=True), 29),       # ... of two segments
    (2, dict(batch=2, hidden=2056, ffn=4104, vocab=1003), 200),
    (2, dict(batch=2, hidden=272, ffn=0, n_experts=16, top_k=4, expert_ffn=136), 24),
    (12, dict(batch=2, hidden=1024, ffn=2040, vocab=2003), 13),                        # short rows, packed
]


def _logits(s, model, opts):
    model.reset_kv()
    dec = GpuDecoder(s, model=model, fusion=31, transitive_reduction=1, **opts)
    out = [dec.step(G.tokens(i, s), np.array([61 + i + 30 * b for b in range(s.batch)], np.int32)) for i in range(3)]
    stats, packed = dec.graph.stats(), int(dec.graph.task_forms()["packed"].max())
    dec.close()
    return np.array(out), stats, packed


@pytest.mark.parametrize("batch_class,kw,workers", SETS)
def test_plain_hybrid_and_per_operator_launches_agree_to_the_bit(batch_class, kw, workers):
    s = G.small_variant("C1", **kw)
    model = DeviceModel(s, 1)
    want, stats, packed = _logits(s, model, dict(n_workers=workers, launch_mode=M.binding.LAUNCH_PER_OP))
    assert np.isfinite(want).all()
    large = s.batch == 1 and stats["weight_bytes"] // s.n_layers // workers >= 3 << 20
    assert batch_class == (9 if large else s.batch + (10 if packed > 1 and not s.n_experts else 0))
    for opts in (dict(), dict(n_sched_wgs=1), dict(n_sched_wgs=2)):
        for debug in (0, M.binding.DEBUG_JITTER):
            got, stats, _ = _logits(s, model, dict(n_workers=workers, debug_flags=debug, **opts))
            assert (stats["n_jit_tasks"] > 0) == ("n_sched_wgs" in opts)
            assert np.array_equal(got, want), (opts, debug)
