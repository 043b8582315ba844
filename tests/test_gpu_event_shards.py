"""Sharded event counters and the static scratch array: a graph whose scratch fits the array only
with its narrow events unsharded still runs from it, and both forms give the step's logits."""
import numpy as np
import pytest
import torch

import paper_2512_22219_amd as M
from synth import gen as G
from synth.device import DeviceModel

LINES = 17 * 256   # bytes of one sharded event's counters


@pytest.mark.gpu
@pytest.mark.parametrize("n_layers,all_sharded", [(300, True), (700, False)])
def test_deep_graphs_keep_the_static_scratch_entry_point(n_layers, all_sharded):
    s = G.small_variant("C1", batch=4, n_layers=n_layers, max_seq=136)
    model = DeviceModel(s, 3)
    graph = M.compile_graph(s, model.weight_ptrs(), model.kv_ptrs(), fusion=31, transitive_reduction=1)
    ex, act = graph.export(), graph.stats()["act_bytes"]
    need = graph.static_scratch_need()
    assert need <= 32 << 20
    assert (need >= act + LINES * (len(ex.events) - 1)) == all_sharded   # (the start event has no producers)
    tok = torch.as_tensor(G.tokens(3, s), device=model.device)
    pos = torch.as_tensor(G.kv_lengths(3, s), device=model.device)
    stream = torch.cuda.current_stream().cuda_stream
    got = []
    for step in (graph.decode_step, graph.decode_step_static, graph.decode_step, graph.decode_step_static):
        lg = torch.full((s.batch, s.vocab), float("nan"), dtype=torch.float32, device=model.device)
        step(tok.data_ptr(), pos.data_ptr(), lg.data_ptr(), stream)
        got.append(lg)
    torch.cuda.synchronize()
    graph.status()
    graph.destroy()
    ref = got[0].cpu().numpy()
    assert np.isfinite(ref).all()
    assert all(np.array_equal(ref, g.cpu().numpy()) for g in got[1:])
