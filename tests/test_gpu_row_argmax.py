"""The rows' arg-max on either side of the size from which it is a kernel of its own (32768 candidates: one for each row
and 16 tokens), against the logits of the same step; ties go to the lowest token."""
import numpy as np
import pytest

import pv_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,rows", [(8192, 64), (8208, 64), (16384, 33), (128256, 4), (128256, 5)])
def test_prediction_is_the_argmax_of_the_logits(vocab, rows):
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    shape = pv_inputs.ModelShape("am_%d" % vocab, 1, 128, 4, 2, 32, 128, vocab, seed=7301)
    gm = gpu_model(shape, max_gamma=64)
    # the last 16 tokens repeat the first 16: every maximum among those has a twin
    head = pv_inputs.fill_tensor(shape, "lm_head", 0).reshape(vocab, shape.d_model).copy()
    head[-16:] = head[:16]
    step = gm.chunk_rows(shape.d_model)
    for r0 in range(0, vocab, step):
        gm.load_weights("lm_head", 0, r0, head[r0:r0 + step])
    c = pv.Cache(gm, 128)
    c.prefill(pv_inputs.uniform_tokens(5, 9, vocab))
    for _ in range(2):
        c.verify(9, np.full(rows, (c.pending + 1) % vocab, dtype=np.int32))
        assert np.array_equal(c.debug_pred(), np.argmax(c.debug_logits(), axis=1))
    c.prefill(pv_inputs.uniform_tokens(6, 100, vocab))
    assert c.debug_pred()[-1] == np.argmax(c.debug_logits()[-1]) == c.pending
