"""Matrix-core linear bodies to the last bit where the lanes that share a row's split into three terms hold the ends of
things: inputs that end inside a k-group of 64 or a chunk, row counts that fill none of a packing's columns, tiles of a few
rows, experts of one to several tokens.  The digests are of the library whose lanes each split all of their row."""
import pytest

from tests.test_gpu_same_bits import digest

pytestmark = pytest.mark.gpu

CASES = [
    (dict(batch=3, hidden=264, ffn=1000, vocab=1003), "02aa5e96348a05a9"),   # three terms in one multiply
    (dict(batch=4, hidden=2056, ffn=520), "96518b9500376f38"),
    (dict(batch=5, hidden=328, ffn=4104, vocab=1003), "26845a1051ce0e5d"),   # two, and a second chunk of 8 inputs
    (dict(batch=7, hidden=4168, ffn=264), "69194d440de7b413"),
    (dict(batch=11, hidden=2056, ffn=712, vocab=1003), "ce45b7d624d568e4"),  # one
    (dict(batch=16, hidden=264, ffn=2120), "c7d1958f3eacacd0"),
    (dict(batch=2, hidden=272, ffn=0, n_experts=16, top_k=4, expert_ffn=136), "25c0e3f2e5ee17fb"),
    (dict(batch=6, hidden=528, ffn=0, n_experts=16, top_k=8, expert_ffn=200), "503e0a09d1c2c387"),
    (dict(batch=12, hidden=1040, ffn=0, n_experts=60, top_k=4, expert_ffn=328), "607a3ca2ead3d0eb"),
]


@pytest.mark.parametrize("kw,want", CASES)
def test_logits_to_the_bit(kw, want):
    assert digest(kw) == want
