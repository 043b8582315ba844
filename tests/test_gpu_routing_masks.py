"""Routing by bit masks: experts that fill no word, end inside one, or need all eight, and one to sixteen chosen of them.  A wrong
choice, count, list or weight moves the logits; the digests are of the library that scanned over the experts."""
import pytest

from tests.test_gpu_same_bits import digest

pytestmark = pytest.mark.gpu

CASES = [   # batch, experts, chosen
    (1, 8, 1, "92de8eadae3b0bf9"),
    (5, 60, 8, "6d7e10c48e212b41"),
    (16, 64, 16, "0164782934b554fc"),
    (2, 72, 4, "bd26ecf92b02f408"),
    (9, 128, 8, "fbfb97bbc5bac262"),
    (16, 136, 3, "14e14eaadadcda6e"),
    (8, 512, 16, "a748fa4ae27ba8ac"),
    (3, 448, 2, "2387f5beede5f336"),
    (16, 512, 16, "48fee2fc1cf4a5a0"),
    (13, 300, 5, "8bff2920558640b0"),
    (16, 129, 8, "07ca53b36a2cfc96"),
    (1, 512, 1, "678a3b3668081847"),
]


@pytest.mark.parametrize("batch,experts,top_k,want", CASES)
def test_logits_to_the_bit(batch, experts, top_k, want):
    assert digest(dict(batch=batch, hidden=272, ffn=0, n_experts=experts, top_k=top_k, expert_ffn=64, vocab=1003)) == want
