"""Rounding of the attention task against 64 bits, with scores large enough that they decide the error of the
logits: an error e of a score (in natural units) is a relative error e of its weight."""
import numpy as np
import pytest
import torch

from oracle import decoder as D
from synth import gen as G
from tests.gpu_util import GpuDecoder, held_step

pytestmark = pytest.mark.gpu
# A score is 64 or 128 exact products.  Summed pairwise, 32 inputs at a time, in 32 bits the root mean square over
# these inputs is 0.75 .. 0.94e-6 (0.88 .. 0.99e-6 in the eight-input runs of a vector body); one accumulator
# for the whole score gives 1.15 .. 1.53e-6 with a head size of 128.
BOUND = 1.05e-6


@pytest.mark.parametrize("head_dim,grp", [(64, 1), (64, 4), (64, 8), (128, 2), (128, 4), (128, 8)])
def test_scores_keep_their_precision(head_dim, grp):
    errs = []
    for seed in range(24):
        s = G.small_variant("C1", n_layers=1, hidden=1024, ffn=128, vocab=512, head_dim=head_dim, n_q_heads=4 * grp,
                            n_kv_heads=4, max_seq=1040)
        ref = D.DecoderOracle(s, G.SynthWeights(s, seed), "f64")
        gpu = GpuDecoder(s, seed, fusion=31, transitive_reduction=1)
        gpu.model.k *= 32.0   # (a power of two: the rows stay bf16 values)
        torch.cuda.synchronize()
        ref._kv(0)[0][...] = gpu.model.k[0].view(torch.int16).cpu().numpy().view(np.uint16)
        got, want, _, _ = held_step(ref, gpu, G.tokens(seed, s), np.array([1020 + seed % 16], np.int32))
        errs.append(float(np.linalg.norm(got - want) / np.linalg.norm(want)))
        gpu.close()
    assert np.sqrt(np.mean(np.square(errs))) < BOUND, errs
