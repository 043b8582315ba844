"""The matrix-core attention task at the edges of its 32-row blocks (8 wavefronts, a block each per
round), for every head size and number of query heads per KV head, and the matrix-core linear task
whose weight rows exceed one job.  Bounds: those of strict_steps (held bf16 decisions, fp64 oracle)."""
import numpy as np
import pytest

from synth import gen as G
from tests.test_gpu_parity import strict_steps

pytestmark = pytest.mark.gpu
FUSED = dict(fusion=31, transitive_reduction=1)
EDGES = [[0, 1, 31], [32, 33, 64], [255, 256, 257], [288, 511, 520]]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("grp", [1, 2, 4, 8])
@pytest.mark.parametrize("opts", [dict(attn_chunks=1, **FUSED),          # blocks wrap around the wavefronts
                                  dict(attn_chunks=17, **FUSED),         # more partials than one merge batch holds
                                  dict(attn_chunks=2, fusion=15),        # RoPE and the append in an operator of their own
                                  dict(attn_chunks=3, fusion=23, launch_mode=1)])   # merge operator
def test_attention_blocks(head_dim, grp, opts):
    s = G.small_variant("C1", n_layers=1, hidden=128, ffn=128, vocab=256, head_dim=head_dim, n_q_heads=2 * grp,
                        n_kv_heads=2, batch=3, max_seq=528)
    for pos in EDGES:
        strict_steps(s, 3, opts, G.tokens(3, s), np.array(pos, np.int32), 1)


@pytest.mark.parametrize("length", [0, 31, 32, 33, 256, 257, 520])
@pytest.mark.parametrize("grp,qk_norm", [(4, False), (8, True)])
def test_attention_blocks_batch_1(length, grp, qk_norm):
    s = G.small_variant("C1", n_layers=2, hidden=128, ffn=128, vocab=256, head_dim=128, n_q_heads=grp, n_kv_heads=1,
                        max_seq=528, qk_norm=qk_norm)
    strict_steps(s, 4, FUSED, G.tokens(4, s), np.array([length], np.int32), 2)


@pytest.mark.parametrize("batch,opts", [(3, dict(tiles_linear=1, tiles_lm_head=1)), (4, dict(tiles_linear=2, tiles_lm_head=1)),
                                        (4, dict(tiles_linear=1, tiles_lm_head=1, launch_mode=1))])
def test_linear_tasks_of_more_rows_than_a_job(batch, opts):
    """One tile per operator: 1376 gate/up rows and 1024 logits a task, in jobs of 512 rows."""
    s = G.small_variant("C1", batch=batch, n_layers=2)
    pos = np.array([3, 77, 150, 20][:batch], np.int32)
    strict_steps(s, 6, dict(n_workers=5, **FUSED, **opts), G.tokens(6, s), pos, 2)


def test_wide_batch_4_inputs_stay_refused_where_the_vector_body_could_not_hold_them():
    import paper_2512_22219_amd as M
    from synth.device import DeviceModel
    s = G.small_variant("C1", batch=4, n_layers=1, ffn=12288)
    model = DeviceModel(s, 0)
    with pytest.raises(M.MpkError) as e:
        M.compile_graph(s, model.weight_ptrs(), model.kv_ptrs(), **FUSED)
    assert e.value.status == M.binding.MPK_ERR_UNSUPPORTED and "LDS" in str(e.value)
