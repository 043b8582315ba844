"""Vector linear bodies (batch 1 and 2) to the last bit on rows that end inside a half block: its stages of 512 inputs past the
row's end are neither requested nor multiplied, one, two or four at a time.  The digests are of the library that multiplied
all of them by zeros."""
import pytest

from tests.test_gpu_same_bits import digest

pytestmark = pytest.mark.gpu

# (inputs of the attention and head projections, of the down projection), digests at batch 1 and 2
CASES = [
    ((8, 504), ("bc2521eba5924f6b", "aaa2de9dca4ef4ce")),
    ((512, 520), ("a9ce50ec969a0fba", "de9a0bb57661123f")),
    ((1024, 1032), ("f0c633b796cf5dc6", "6b249ad3e3e11a78")),
    ((1544, 2048), ("83b42c9815d06fa8", "48d24a211179047a")),
    ((2056, 3584), ("00da1f3b25227625", "83f339c5bd44f7d3")),
    ((3592, 4104), ("80cf2c0a222779a9", "b672b297a50ff0e9")),
    ((4608, 6152), ("11b9aa8b8439b634", "738549b1926c6a49")),
]


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("sizes,want", CASES)
def test_logits_to_the_bit(sizes, want, batch):
    kw = dict(batch=batch, hidden=sizes[0], ffn=sizes[1], vocab=1003)
    if sizes[0] == 8:
        kw["max_seq"] = 64
    assert digest(kw) == want[batch - 1]
