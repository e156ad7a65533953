"""Attention of short contexts (up to two chunks of keys: one workgroup per kv head goes through them, no merge) against the
oracle, on both sides of the limits: 512 keys with up to 16 query rows per kv head, 256 with more."""
import numpy as np
import pytest

import pv_inputs
from helpers import ref_model
from oracle import ref

pytestmark = pytest.mark.gpu

S = pv_inputs.ModelShape
SHAPES = {"gqa": S("sc_gqa", 2, 256, 8, 2, 64, 704, 512, rope_base=500000.0, seed=7201), "mha": S("sc_mha", 2, 256, 2, 2, 128, 704, 512, seed=7202),
          "hd32": S("sc_hd32", 2, 128, 12, 4, 32, 352, 512, seed=7203)}


@pytest.mark.parametrize("name,prefix,rows", [("gqa", 1, 1), ("gqa", 17, 4), ("gqa", 250, 4), ("gqa", 253, 4), ("gqa", 505, 4), ("gqa", 509, 4),
                                              ("gqa", 120, 8), ("gqa", 121, 8), ("gqa", 248, 8), ("gqa", 249, 8), ("gqa", 100, 64), ("gqa", 192, 64),
                                              ("mha", 300, 16), ("mha", 240, 16), ("mha", 222, 33), ("hd32", 400, 5), ("hd32", 130, 6), ("hd32", 0, 40)])
def test_short_context(name, prefix, rows):
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model, logit_scale
    shape = SHAPES[name]
    gm = gpu_model(shape, gains="perturbed", max_gamma=64)
    rc = ref.RefCache(ref_model(shape, gains="perturbed"), 640, ref.KV_BF16)
    toks = pv_inputs.uniform_tokens(81, prefix + rows, shape.vocab)
    graph, plain = pv.Cache(gm, 640), pv.Cache(gm, 640)
    plain.use_graphs(False)
    if prefix:
        rc.prefill(toks[:prefix])
    _, _, _, want = rc.verify(prefix, toks[prefix:], want_logits=True)
    for c in (graph, plain):
        if prefix:
            c.prefill(toks[:prefix])
        c.verify(prefix, toks[prefix:])
        assert (np.abs(c.debug_logits() - want) / logit_scale(want)).max() < 2e-3
