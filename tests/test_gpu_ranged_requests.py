"""Matrix-core linear tasks whose rounds hold few real weight fragments -- the rest of a round is loads past the
range of the buffer -- and inputs that end inside a 64-input group, with the look at the event ahead of the requests
and without pre-loading; and the routing of few and of many experts.  Bounds: those of strict_steps (held
bf16 decisions, fp64 oracle)."""
import numpy as np
import pytest

from synth import gen as G
from tests.test_gpu_parity import strict_steps

pytestmark = pytest.mark.gpu
FUSED = dict(fusion=31, transitive_reduction=1)


@pytest.mark.parametrize("batch", [3, 5, 8, 9, 16])
@pytest.mark.parametrize("hidden,ffn", [(128, 136),     # two k-groups: most slots of a round are empty
                                        (264, 72),      # eight inputs into a group
                                        (2056, 2120)])  # a chunk and eight inputs (batch above 8)
@pytest.mark.parametrize("opts", [dict(), dict(no_preload=1), dict(tiles_linear=9, n_workers=7)])
def test_rounds_with_few_fragments(batch, hidden, ffn, opts):
    s = G.small_variant("C1", n_layers=2, hidden=hidden, ffn=ffn, vocab=200, batch=batch, max_seq=64)
    pos = (np.arange(batch) * 5 % 61).astype(np.int32)
    strict_steps(s, 5, dict(**FUSED, **opts), G.tokens(5, s), pos, 2)


@pytest.mark.parametrize("n_experts,top_k", [(64, 1), (72, 7), (128, 8), (136, 9), (200, 16)])   # both routing bodies; a combine round of eight and a part of one
@pytest.mark.parametrize("batch", [1, 3, 16])
def test_routing_and_combine(n_experts, top_k, batch):
    s = G.small_variant("C1", n_layers=2, hidden=128, ffn=0, vocab=256, batch=batch, max_seq=64, n_experts=n_experts,
                        top_k=top_k, expert_ffn=40)
    pos = (np.arange(batch) * 7 % 61).astype(np.int32)
    strict_steps(s, 8, FUSED, G.tokens(8, s), pos, 2)
