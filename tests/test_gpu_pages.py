"""Pre-load pages in LDS: where a task finds its first weight rows must not show in the logits."""
import numpy as np
import pytest

from synth import gen as G
from synth.device import DeviceModel
from tests.gpu_util import GpuDecoder
from tests.test_compiler import PAGE_CHAINS, RESIZED

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,workers", PAGE_CHAINS + [(dict(hidden=512, ffn=12288), 29), (dict(hidden=2048, n_q_heads=16, ffn=8192), 24),
                                                      (dict(hidden=2048, n_q_heads=16, ffn=4096), 24)])
def test_logits_with_pages_equal_those_without(kw, workers):
    _compare(kw, dict(fusion=31, transitive_reduction=1, n_workers=workers))


@pytest.mark.parametrize("kw,opts", RESIZED)
def test_logits_where_the_tile_sizes_change_the_graph(kw, opts):
    _compare(kw, opts)


def _compare(kw, opts):
    s = G.small_variant("C1", **kw)
    model, out = DeviceModel(s, 1), []
    for off in (0, 1):
        model.reset_kv()
        dec = GpuDecoder(s, model=model, no_lds_pages=off, **opts)
        out.append([dec.step(G.tokens(i, s), np.array([61 + i], np.int32)) for i in range(3)])
        dec.close()
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1])
