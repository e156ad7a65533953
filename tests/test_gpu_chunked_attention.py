"""Attention in chunks of keys with a merge behind it, against the oracle, where the cache's length falls on the edges of what a wave takes (32 keys: all committed, part of the
block among them, the second group of 16 past the end) and of a chunk, with query rows that fill a tile of 16 and rows that do not."""
import numpy as np
import pytest

import pv_inputs
from helpers import ref_model
from oracle import ref

pytestmark = pytest.mark.gpu

S = pv_inputs.ModelShape
SHAPES = {"gqa": S("ca_gqa", 1, 256, 8, 2, 64, 352, 512, rope_base=500000.0, seed=7301), "mha": S("ca_mha", 1, 256, 2, 2, 128, 352, 512, seed=7302),
          "group3": S("ca_g3", 1, 128, 12, 4, 32, 352, 512, seed=7303), "pages16": S("ca_p16", 1, 256, 4, 2, 128, 352, 512, seed=7304).replace(page_tokens=16)}


@pytest.mark.parametrize("name,prefix,rows", [("gqa", 767, 1), ("gqa", 768, 4), ("gqa", 765, 4), ("gqa", 287, 8), ("gqa", 288, 8), ("gqa", 600, 13), ("mha", 543, 16),
                                              ("mha", 544, 3), ("mha", 1008, 33), ("group3", 575, 5), ("group3", 608, 6), ("group3", 576, 40), ("pages16", 640, 8), ("pages16", 303, 9)])
def test_chunks_of_keys(name, prefix, rows):
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model, logit_scale
    shape = SHAPES[name]
    gm = gpu_model(shape, gains="perturbed", max_gamma=64)
    rc = ref.RefCache(ref_model(shape, gains="perturbed"), 1152, ref.KV_BF16)
    toks = pv_inputs.uniform_tokens(83, prefix + rows, shape.vocab)
    rc.prefill(toks[:prefix])
    _, _, _, want = rc.verify(prefix, toks[prefix:], want_logits=True)
    c = pv.Cache(gm, 1152)
    pages = -(-1152 // shape.page_tokens)
    c.set_page_table(np.random.default_rng(3).permutation(pages).astype(np.int32))
    c.prefill(toks[:prefix])
    c.verify(prefix, toks[prefix:])
    assert (np.abs(c.debug_logits() - want) / logit_scale(want)).max() < 2e-3
