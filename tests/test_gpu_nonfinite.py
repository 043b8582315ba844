"""Infinite elements.  In the cache: a row whose score is -infinity has weight 0 and leaves the step's logits as
finite as they are without it; an infinite value gives NaN in its own sequence and nowhere else.  In a weight, up
to four sequences: an infinite output of that row.  Bounds: those of strict_steps (held bf16 decisions, fp64 oracle)."""
import numpy as np
import pytest
import torch

import paper_2512_22219_amd as M
from oracle import decoder as D
from synth import gen as G
from synth.device import DeviceModel
from tests.gpu_util import GpuDecoder, appended_rows, bf16_bits_to_f64, held_step, rel_err

pytestmark = pytest.mark.gpu
FUSED = dict(fusion=31, transitive_reduction=1)
PLUS, MINUS = 0x7F80, 0xFF80


def _queries(s, w, tok, pos):
    """The first query head of each KV group after the rotation, [B][n_kv][d] (layer 0, 64 bits)."""
    l0, d, grp = w.layer(0), s.head_dim, s.n_q_heads // s.n_kv_heads
    out = np.zeros((s.batch, s.n_kv_heads, d))
    for b in range(s.batch):
        x = bf16_bits_to_f64(w.embed_row(int(tok[b])))
        h = x / np.sqrt(np.mean(x * x) + s.rms_eps) * bf16_bits_to_f64(l0[G.L_ATTN_NORM]).ravel()
        for g in range(s.n_kv_heads):
            q = bf16_bits_to_f64(l0[G.L_WQKV][g * grp * d:(g * grp + 1) * d]) @ h
            a = pos[b] * float(s.rope_theta) ** (-2.0 * np.arange(d // 2) / d)
            lo, hi = q[:d // 2], q[d // 2:]
            out[b, g] = np.concatenate([lo * np.cos(a) - hi * np.sin(a), hi * np.cos(a) + lo * np.sin(a)])
    return out


def _run(s, seed, pos, mark_k, mark_v, page=0, **opts):
    """One step with K rows mark_k[b] of sequence b giving -infinity as score for every head, and V rows
    mark_v[b] holding an infinity: (GPU logits, oracle logits)."""
    w = G.SynthWeights(s, seed)
    d, grp = s.head_dim, s.n_q_heads // s.n_kv_heads
    wqkv = w.layer(0)[G.L_WQKV]
    for h in range(s.n_q_heads):      # the heads of a group alike: one sign of every query element
        g = h // grp * grp
        wqkv[h * d:(h + 1) * d] = wqkv[g * d:(g + 1) * d]
    tok, pos = G.tokens(seed, s), np.array(pos, np.int32)
    q = _queries(s, w, tok, pos)
    model, ref = DeviceModel(s, seed), D.DecoderOracle(s, w, "f64")
    model.layers[0]["wqkv"].copy_(torch.from_numpy(wqkv.view(np.int16)).view(torch.bfloat16))
    K, V = ref._kv(0)
    for b in range(s.batch):
        for g in range(s.n_kv_heads):
            e = int(np.abs(q[b, g]).argmax())
            for r in mark_k.get(b, []):
                K[b, g, r, e] = MINUS if q[b, g, e] > 0 else PLUS
            for r in mark_v.get(b, []):
                V[b, g, r, 3] = PLUS
    dev = model.device

    def up(a):
        return torch.from_numpy(a.view(np.int16).copy()).to(dev).view(torch.bfloat16)

    model.k[0].copy_(up(K))
    model.v[0].copy_(up(V))
    if page:
        n_pages = s.batch * (s.max_seq // page) + 3
        table = G.page_table(seed, s, page, n_pages, pos + 1)
        pools = [up(G.paginate(c, table, page, n_pages))[None].contiguous() for c in (K, V)]
        g = M.compile_graph(s, model.weight_ptrs(), tuple(p.data_ptr() for p in pools), kv_page_size=page, kv_pages=n_pages, **opts)
        d_table = torch.as_tensor(table, device=dev)
        g.set_page_table(d_table.data_ptr())
    else:
        g = M.compile_graph(s, model.weight_ptrs(), model.kv_ptrs(), **opts)
    t, p = torch.as_tensor(tok.astype(np.int32), device=dev), torch.as_tensor(pos, device=dev)
    lg = torch.zeros((s.batch, s.vocab), dtype=torch.float32, device=dev)
    g.decode_step(t.data_ptr(), p.data_ptr(), lg.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    g.status()
    if page:
        rows = [np.stack([pool[0].view(torch.int16).cpu().numpy().view(np.uint16)[table[b, pos[b] // page], :, pos[b] % page]
                          for b in range(s.batch)])[None] for pool in pools]
    else:
        rows = appended_rows(model, pos)
    g.destroy()
    with np.errstate(all="ignore"):
        want = ref.step(tok, pos, held=D.Held(rows[0], rows[1], None))
    return lg.cpu().numpy(), want


SHAPES = [(64, 1), (64, 4), (64, 8), (128, 2), (128, 8)]


@pytest.mark.parametrize("head_dim,grp", SHAPES)
@pytest.mark.parametrize("opts", [dict(attn_chunks=3, no_attn_balance=1), dict(attn_chunks=1), dict(attn_chunks=2, page=16),
                                  dict(attn_chunks=3, no_attn_balance=1, fusion=23), dict(attn_chunks=2, no_attn_balance=1, launch_mode=1)])
def test_rows_of_weight_zero(head_dim, grp, opts):
    s = G.small_variant("C1", n_layers=1, hidden=256, ffn=128, vocab=256, head_dim=head_dim, n_q_heads=2 * grp, n_kv_heads=2,
                        batch=2, max_seq=544)
    marks = {0: list(range(0, 40)) + [77, 300],      # the first block of a wavefront, and single rows
             1: list(range(0, 180)) + [511]}         # a whole chunk (of 531 rows in three)
    got, want = _run(s, 5, [400, 530], marks, {}, **{**FUSED, **opts})
    assert np.isfinite(want).all()
    assert np.isfinite(got).all()
    assert rel_err(got, want) < 2e-2
    assert np.abs(got - want).max() / np.abs(want).max() < 2e-5


@pytest.mark.parametrize("head_dim,grp", SHAPES)
def test_an_infinite_value_stays_in_its_sequence(head_dim, grp):
    s = G.small_variant("C1", n_layers=1, hidden=256, ffn=128, vocab=256, head_dim=head_dim, n_q_heads=2 * grp, n_kv_heads=2,
                        batch=2, max_seq=544)
    got, want = _run(s, 6, [400, 530], {1: [40]}, {0: [100]}, **FUSED)
    assert not np.isfinite(got[0]).any() and np.isfinite(got[1]).all()
    assert np.abs(got[1] - want[1]).max() / np.abs(want[1]).max() < 2e-5


@pytest.mark.parametrize("batch", [1, 2, 3, 4])
@pytest.mark.parametrize("opts", [dict(), dict(launch_mode=1)])
def test_an_infinite_weight_gives_an_infinite_logit(batch, opts):
    """One element of three rows of the output head, two of a fourth (not among a row's last eight, which are also
    multiplied with the zeros behind it)."""
    s = G.small_variant("C1", n_layers=1, hidden=264, ffn=128, vocab=300, batch=batch, max_seq=64)
    w = G.SynthWeights(s, 9)
    head = w.lm_head()
    for row, cols in ((0, [(5, PLUS)]), (17, [(255, MINUS)]), (299, [(0, PLUS)]), (150, [(1, PLUS), (200, PLUS)])):
        for c, bits in cols:
            head[row, c] = bits
    gpu = GpuDecoder(s, 9, **{**FUSED, **opts})
    gpu.model.lm_head.copy_(torch.from_numpy(head.view(np.int16)).view(torch.bfloat16))
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        got, want, _, _ = held_step(D.DecoderOracle(s, w, "f64"), gpu, G.tokens(9, s), np.arange(batch, dtype=np.int32) * 7 + 3)
    gpu.close()
    assert np.isinf(want[:, [0, 17, 299]]).all()
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    inf, fin = np.isinf(want), np.isfinite(want)
    assert np.array_equal(got[inf], want[inf])
    assert np.abs(got[fin] - want[fin]).max() / np.abs(want[fin]).max() < 2e-5
