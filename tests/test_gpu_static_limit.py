"""A step whose buffers just fit the fixed array of pv_verify_async_static: only what the kernels use is counted."""
import numpy as np
import pytest

import pv_inputs

pytestmark = pytest.mark.gpu

# fp32, 64 rows: 31.9 of 32 MiB, half a MiB more with separate buffers for normed rows, keys and values
WIDE = pv_inputs.ModelShape("sl_wide", 1, 64, 8, 8, 128, 64, 128000, dtype="f32", seed=7601)


def test_a_step_that_just_fits():
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    gm = gpu_model(WIDE, gains="perturbed", max_gamma=64)
    a, b = pv.Cache(gm, 128), pv.Cache(gm, 128)
    prompt, draft = pv_inputs.uniform_tokens(1, 20, WIDE.vocab), pv_inputs.uniform_tokens(2, 64, WIDE.vocab)
    a.prefill(prompt); b.prefill(prompt)
    draft[0] = a.pending
    want = a.verify(20, draft)
    b.verify_async_static(20, draft)
    assert b.verify_wait() == want and np.array_equal(a.export(), b.export())
