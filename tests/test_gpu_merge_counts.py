"""The merge of a sequence's attention partials for every number of them: they are loaded eight, four, two and one at a time,
sixteen to a round.  The marked launch merges all but its own partial from memory, the per-operator launch all of them, in the same
order: equal to the last bit.  One chunk, which merges nothing, is the reference for both; chunks change the order of
additions only, and what that does to logits of size one is some 2 ** -24 an addition over a few hundred of them."""
import numpy as np
import pytest
import torch

import paper_2512_22219_amd as M
from synth import gen as G
from synth.device import DeviceModel

pytestmark = pytest.mark.gpu


def _step(s, model, **opts):
    model.reset_kv()
    g = M.compile_graph(s, model.weight_ptrs(), model.kv_ptrs(), fusion=31, transitive_reduction=1, **opts)
    tok = torch.as_tensor(G.tokens(3, s).astype(np.int32), device=model.device)
    pos = torch.as_tensor(np.array([s.max_seq - 3 - 50 * b for b in range(s.batch)], np.int32), device=model.device)
    out = torch.empty((s.batch, s.vocab), dtype=torch.float32, device=model.device)
    g.decode_step(tok.data_ptr(), pos.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    g.status()
    g.destroy()
    return out.cpu().numpy()


@pytest.mark.parametrize("kw", [dict(), dict(batch=2, head_dim=128, n_q_heads=8, n_kv_heads=1), dict(batch=3)])
def test_every_number_of_partials(kw):
    s = G.small_variant("C1", max_seq=320, **kw)
    model = DeviceModel(s, 1)
    one = _step(s, model, attn_chunks=1)
    for chunks in list(range(2, 20)) + [24, 33]:
        got, ref = _step(s, model, attn_chunks=chunks), _step(s, model, attn_chunks=chunks, launch_mode=1)
        assert np.array_equal(got, ref), chunks
        assert np.abs(got - one).max() < 2e-5 * np.abs(one).max(), chunks
