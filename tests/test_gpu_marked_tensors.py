"""Marked activation tensors (batch 1 and 2): a consumer loads its input until no word of it is unset, instead of
waiting for an event, and every step puts the other step's copy back to unset.

The per-operator launches and the one launch of the loop kernel run the same task bodies on unmarked descriptors
and on memory of their own, and the arithmetic does not depend on how a task learns that its input is
complete: logits have to be equal to the last bit, step after step (a word taken before it was written, or one of
the step before last that was not put back, shows)."""
import numpy as np
import pytest
import torch

import paper_2512_22219_amd as M
from synth import gen as G
from synth.device import DeviceModel

pytestmark = pytest.mark.gpu
FUSED = dict(fusion=31, transitive_reduction=1)


def _greedy(s, model, n, calls=None, **opts):
    dev = model.device
    model.reset_kv()
    g = M.compile_graph(s, model.weight_ptrs(), model.kv_ptrs(), **opts)
    marked = bool((g.task_forms()["marks"] & M.binding.FORM_INPUT_MARKED).any())
    assert marked == (opts.get("launch_mode", 0) == 0 and opts["greedy_loop"] != 2)   # (or a comparison says nothing)
    tok = torch.as_tensor(G.tokens(3, s).astype(np.int32), device=dev)
    pos = torch.as_tensor(np.array([(37 * b + 61) % (s.max_seq - n) for b in range(s.batch)], np.int32), device=dev)
    picked = torch.empty((n, s.batch), dtype=torch.int32, device=dev)
    logits = torch.empty((s.batch, s.vocab), dtype=torch.float32, device=dev)
    every = torch.empty((n, s.batch, s.vocab), dtype=torch.float32, device=dev)
    at = 0
    for k in calls or [n]:
        g.decode_steps(k, tok.data_ptr(), pos.data_ptr(), picked[at].data_ptr(), logits.data_ptr(), every[at].data_ptr(), torch.cuda.current_stream().cuda_stream)
        at += k
    torch.cuda.synchronize()
    g.status()
    g.destroy()
    return every.cpu().numpy(), picked.cpu().numpy()


SHAPES = [
    dict(),                                                         # one slice of the input, one chunk of rows
    dict(batch=2),
    dict(hidden=2056, ffn=4104, vocab=1003),                        # a slice and 8 inputs; a 4096-input segment and 8
    dict(hidden=512, ffn=12296, batch=2),                           # 12288 inputs a round trip, and 8
    dict(hidden=256, ffn=28672),                                    # three round trips
    dict(hidden=2048, n_q_heads=16, n_kv_heads=2, max_seq=2624),    # 20 chunk tasks a head: two blocks of the merge
    dict(hidden=1024, n_q_heads=8, n_kv_heads=1, head_dim=128, qk_norm=True, max_seq=1024),
    dict(n_experts=16, top_k=4, ffn=0, expert_ffn=64),
]


@pytest.mark.parametrize("debug", [0, 4])   # 4: every task starts after a pseudo-random delay
@pytest.mark.parametrize("kw", SHAPES)
def test_marked_launches_equal_unmarked_ones(kw, debug):
    s = G.small_variant("C1", **kw)
    model, n = DeviceModel(s, 1), 5
    want, tokens = _greedy(s, model, n, greedy_loop=1, launch_mode=1, **FUSED)
    got, picked = _greedy(s, model, n, greedy_loop=1, debug_flags=debug, **FUSED)
    assert np.isfinite(want).all() and np.array_equal(got, want) and np.array_equal(picked, tokens)
    loop, _ = _greedy(s, model, n, greedy_loop=2, **FUSED)
    assert np.array_equal(loop, want)
    few, _ = _greedy(s, model, n, greedy_loop=1, n_workers=29, **FUSED)   # several tasks of an operator per worker
    ref, _ = _greedy(s, model, n, greedy_loop=1, launch_mode=1, n_workers=29, **FUSED)
    assert np.array_equal(few, ref)


@pytest.mark.parametrize("kw,opts", [
    (dict(), dict(tiles_linear=2)), (dict(batch=2), dict(tiles_linear=2)), (dict(hidden=512, batch=2), dict(n_workers=15)),
    (dict(n_experts=16, top_k=4, ffn=0, expert_ffn=64), dict(n_workers=11)),
    (dict(n_experts=16, top_k=4, ffn=0, expert_ffn=64, batch=2), dict(tiles_linear=3)),
    (dict(hidden=4096, n_q_heads=16, batch=2), dict(tiles_linear=2)),
])
@pytest.mark.parametrize("debug", [0, 4])
def test_large_tiles_whose_residual_is_not_marked(kw, opts, debug):
    """More outputs a task than wavefronts with input: the residual (an embedding row, another one in every step; a
    combined expert output) must not be read ahead of the operators that write it."""
    s = G.small_variant("C1", **kw)
    model, n = DeviceModel(s, 1), 5
    want, tokens = _greedy(s, model, n, greedy_loop=1, launch_mode=1, **FUSED, **opts)
    got, picked = _greedy(s, model, n, greedy_loop=1, debug_flags=debug, **FUSED, **opts)
    assert np.isfinite(want).all() and np.array_equal(got, want) and np.array_equal(picked, tokens)


@pytest.mark.parametrize("calls", [[1, 3, 1, 2, 1], [1, 2, 1, 1, 3]])
@pytest.mark.parametrize("greedy_loop", [1, 2])
def test_calls_of_one_step_between_calls_of_several(greedy_loop, calls):
    """With greedy_loop = 2 a call of several steps is one launch of the loop kernel, which leaves marked copies alone: a
    copy that a single step wrote would be taken for the output of a step of the same parity behind it."""
    s = G.small_variant("C1", batch=2)
    model, n = DeviceModel(s, 1), sum(calls)
    want, tokens = _greedy(s, model, n, greedy_loop=1, launch_mode=1, **FUSED)
    got, picked = _greedy(s, model, n, calls, greedy_loop=greedy_loop, **FUSED)
    assert np.array_equal(got, want) and np.array_equal(picked, tokens)


@pytest.mark.parametrize("opts", [dict(fusion=31), dict(fusion=15, transitive_reduction=1), dict(fusion=30, transitive_reduction=1),
                                  dict(fusion=29, transitive_reduction=1), dict(fusion=27, transitive_reduction=1)])
def test_graphs_that_mark_only_some_of_their_tensors(opts):
    s = G.small_variant("C1", batch=2)
    model = DeviceModel(s, 1)
    want, _ = _greedy(s, model, 4, greedy_loop=1, launch_mode=1, **opts)
    got, _ = _greedy(s, model, 4, greedy_loop=1, debug_flags=4, **opts)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("after", [1, 2, 3])
def test_steps_skipped_after_the_server_has_drained_leave_both_copies_unset(after):
    """A run that is `after` iterations longer than its requests: the launches behind the drained iteration run no
    task, so nobody but they can put that iteration's copy back.  The next requests must be served as by a
    server that has never drained."""
    s = G.small_variant("C1", batch=2)
    model, stream = DeviceModel(s, 1), torch.cuda.current_stream().cuda_stream

    def serve(first):
        pools = [torch.zeros((s.n_layers, 16, s.n_kv_heads, 32, s.head_dim), dtype=torch.bfloat16, device=model.device) for _ in range(2)]
        g = M.compile_graph(s, model.weight_ptrs(), tuple(p.data_ptr() for p in pools), greedy_loop=1, serving=1, kv_page_size=32, kv_pages=16, **FUSED)
        srv = g.serve(8, 4, 8, -1)
        if first:   # 2 + 3 - 1 iterations of work, one that finds nothing left, `after` that are skipped
            srv.submit([5, 9], 3, stream)
            srv.run(4 + 1 + after, stream)
        ids = [srv.submit(p, 6, stream) for p in ([7, 3, 1], [11, 2])]
        srv.run(9, stream)
        torch.cuda.synchronize()
        g.status()
        out = [srv.result(i) for i in ids]
        g.destroy()
        return out

    assert serve(True) == serve(False)
