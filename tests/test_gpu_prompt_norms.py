"""Long prompts of models whose width is no multiple of what one round of k_pre_rscale, or of its part in k_pre_rowmax (4-bit weights), adds up: 512 and 128 strips of sums of squares."""
import numpy as np
import pytest

import pv_inputs
from helpers import ref_model
from oracle import ref

pytestmark = pytest.mark.gpu

S = pv_inputs.ModelShape
SHAPES = {"16_34": S("pn_34", 1, 544, 4, 2, 64, 256, 512, seed=7851), "16_512": S("pn_512", 1, 8192, 4, 2, 64, 256, 512, seed=7852), "16_516": S("pn_516", 1, 8256, 4, 2, 64, 256, 512, seed=7853),
          "q4_128": S("pn_q128", 1, 2048, 4, 2, 64, 256, 512, seed=7854, weight_bits=4), "q4_136": S("pn_q136", 1, 2176, 4, 2, 64, 256, 512, seed=7855, weight_bits=4)}


@pytest.mark.parametrize("name", SHAPES)
def test_norms_of_a_long_prompt(name):
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model, logit_scale
    shape, n = SHAPES[name], 83
    gm, rm = gpu_model(shape, gains="perturbed"), ref_model(shape, gains="perturbed")
    toks = pv_inputs.uniform_tokens(75, n, shape.vocab)
    c, rc = pv.Cache(gm, n + 16), ref.RefCache(rm, n + 16, ref.KV_BF16)
    c.prefill(toks)
    last = rc.prefill(toks)
    assert (np.abs(c.debug_logits()[-1] - last) / logit_scale(last)).max() < 2e-3       # (as for blocks: bf16 rounding of keys and values)
    got, want = pv_inputs.bf16_bits_to_f32(c.export()).astype(np.float64), rc.export()
    assert np.mean(got != want) < 0.02 and np.abs(got - want).max() <= 2.0 ** -7 * np.abs(want).max()
