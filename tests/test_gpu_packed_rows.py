"""Short weight rows packed two or four to a row of a half block (vector linear body, up to 2048 and 1024 inputs): logits
against the fp64 oracle, at sizes where a half block is full, ends inside a row, ends between rows and lacks its
second row, and where the input ends inside its share."""
import numpy as np
import pytest

import paper_2512_22219_amd as M
from synth import gen as G
from tests.test_gpu_parity import strict_steps

pytestmark = pytest.mark.gpu


def _check(s, packs, opts, tok, pos, steps):
    """`packs`: inputs -> so many weight rows share a row of a half block in some of the graph's tasks of as many inputs."""
    forms = M.compile_graph(s, None, None, host_only=1, **opts).task_forms()
    for inputs, rows in packs.items():
        assert rows in forms["packed"][forms["inputs"] == inputs]
    strict_steps(s, 1, opts, tok, pos, steps)


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("kw,workers,packs", [
    (dict(hidden=2048, ffn=2048, vocab=1000), 29, {2048: 2}),     # two a row, rows that follow one another without a gap
    (dict(hidden=2040, ffn=2056, vocab=1003), 31, {2040: 2, 2056: 1}),     # two a row, the input ends inside; a projection that is not packed
    (dict(hidden=1032, ffn=1024, vocab=997), 15, {1032: 2, 1024: 4}),      # two a row by 8 inputs; four a row
    (dict(hidden=1024, ffn=1024, vocab=2000), 13, {1024: 4}),     # four a row
    (dict(hidden=1000, ffn=520, vocab=1999), 11, {1000: 4, 520: 4}),      # four a row, the input ends inside
    (dict(hidden=256, ffn=688, vocab=1024), 7, {256: 4, 688: 2}),        # the shortest rows
    (dict(hidden=512, ffn=4096, vocab=4093, n_q_heads=8, n_kv_heads=8, qk_norm=True), 7, {512: 4, 4096: 1}),   # (5 workers: large tasks, not packed)
])
def test_packed_rows_match_the_oracle(kw, workers, packs, batch):
    s = G.small_variant("C1", batch=batch, **kw)
    tok = G.tokens(1, s)
    pos = np.array([(41 * b + 7) % 120 for b in range(s.batch)], np.int32)
    _check(s, packs, dict(fusion=31, transitive_reduction=1, n_workers=workers), tok, pos, 2)


@pytest.mark.parametrize("kw,packs", [(dict(hidden=2048, ffn=2048), {2048: 2}), (dict(hidden=1000, ffn=520), {1000: 4})])
def test_packed_rows_with_preloading_off_and_unfused(kw, packs):
    s = G.small_variant("C1", batch=2, **kw)
    tok, pos = G.tokens(1, s), np.array([7, 48], np.int32)
    _check(s, packs, dict(fusion=31, transitive_reduction=1, n_workers=13, no_preload=1), tok, pos, 2)
    _check(s, packs, dict(fusion=7, n_workers=13), tok, pos, 2)
    _check(s, packs, dict(fusion=7, n_workers=13, n_sched_wgs=1), tok, pos, 2)
