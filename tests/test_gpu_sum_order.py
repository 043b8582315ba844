"""The order in which the vector linear body (batch 1 and 2) adds up is part of its results: a last bit of a sum decides
which way an appended bf16 row rounds, and everything behind follows that row.  The widths of its loads and how it
packs its rows must not show, so the order is written out here once and compared to the bit."""
import numpy as np
import pytest
import torch

import paper_2512_22219_amd as M
from synth import gen as G
from synth.device import DeviceModel

pytestmark = pytest.mark.gpu
FUSED = dict(fusion=31, transitive_reduction=1)
f32, f64 = np.float32, np.float64


def _fma(a, b, s):   # one rounding: the inputs below have few enough bits for 64-bit sums to be exact
    return (a.astype(f64) * b.astype(f64) + s.astype(f64)).astype(f32)


def _wave_sum(v):   # [64] -> neighbours, pairs, fours, eights in each row of 16 lanes, then the rows
    while v.size > 4:
        v = v[0::2] + v[1::2]
    return (v[0] + v[1]) + (v[2] + v[3])


def _sum_of_squares(x):
    """A thread takes the pairs of inputs t, t + 512, ... one after the other; wavefronts are added in order."""
    pairs = np.zeros((-(-x.size // 1024) * 512, 2), f32)
    pairs.reshape(-1)[:x.size] = x
    s = np.zeros(512, f32)
    for u in pairs.reshape(-1, 512, 2):
        s = _fma(u[:, 0], u[:, 0], s)
        s = _fma(u[:, 1], u[:, 1], s)
    total = f32(0)
    for w in s.reshape(8, 64):
        total = total + _wave_sum(w)
    return total


def _logits(s, model, tokens, **opts):
    dev = model.device
    g = M.compile_graph(s, model.weight_ptrs(), model.kv_ptrs(), **FUSED, **opts)
    tok = torch.as_tensor(np.asarray(tokens, np.int32), device=dev)
    pos = torch.full((s.batch,), 5, dtype=torch.int32, device=dev)
    out = torch.empty((s.batch, s.vocab), dtype=torch.float32, device=dev)
    g.decode_step(tok.data_ptr(), pos.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    g.status()
    g.destroy()
    return out.cpu().numpy()


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("hidden", [8, 256, 520, 1000, 2048, 4096, 4104, 8192, 12296])   # ... and a second round trip of 12288 inputs
def test_order_of_the_sums_of_squares(hidden, batch):
    """Layers whose output projections are zero leave the embedding row as it is; a head of one-hot rows then shows the
    row's 1 / rms in every logit."""
    s = G.small_variant("C1", hidden=hidden, batch=batch, vocab=256)
    model = DeviceModel(s, 1)
    rng = np.random.default_rng(hidden)
    x = rng.uniform(2.0 ** -6, 4.0, (s.vocab, hidden)) * rng.choice([-1.0, 1.0], (s.vocab, hidden))
    model.embed.copy_(torch.as_tensor(x))
    x = model.embed.float().cpu().numpy()
    model.final_norm.fill_(1.0)
    at = np.arange(s.vocab) * 37 % hidden
    model.lm_head.zero_()
    model.lm_head[torch.arange(s.vocab), torch.as_tensor(at)] = 1.0
    for d in model.layers:
        d["wo"].zero_()
        d["wd"].zero_()
    for i in range(4):
        tokens = rng.integers(0, s.vocab, batch)
        got = _logits(s, model, tokens)
        for b, t in enumerate(tokens):
            inv = f32(1) / np.sqrt(_sum_of_squares(x[t]) / f32(hidden) + f32(s.rms_eps))
            assert np.array_equal(got[b], x[t][at] * inv), (i, b)


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("kw,workers", [
    (dict(hidden=2048, ffn=2048, vocab=1000), 13),    # two rows a half-block row, full
    (dict(hidden=2040, ffn=2056, vocab=1003), 11),    # ... the input ends inside; a projection that is not packed beside it
    (dict(hidden=1032, ffn=8200, vocab=997), 13),     # ... by 8 inputs past four a row; a row of three segments
    (dict(hidden=1024, ffn=1024, vocab=2000), 9),     # four a row, full
    (dict(hidden=256, ffn=688, vocab=1024), 5),       # the shortest rows
])
def test_packed_rows_are_added_up_like_rows_of_their_own(kw, workers, batch):
    """With 256 workers no task has rows enough to be packed, with few all have; every output is a whole row's sum
    either way."""
    s = G.small_variant("C1", batch=batch, **kw)
    model, rng = DeviceModel(s, 1), np.random.default_rng(workers)
    for _ in range(2):
        tokens = rng.integers(0, s.vocab, batch)
        want = _logits(s, model, tokens, n_workers=256, attn_chunks=1)
        got = _logits(s, model, tokens, n_workers=workers, attn_chunks=1)
        assert np.isfinite(want).all() and np.array_equal(got, want)
