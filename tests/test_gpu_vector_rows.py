"""fp32 projections at the edges of what a wavefront takes: groups of 1, 4, 8 and 16 rows and several of 16 in one launch, rows of features in one trip of up to
1024 (512, 256 with more rows), ragged in the last piece and with a second trip, against the oracle."""
import numpy as np
import pytest

import pv_inputs
from helpers import ref_model
from oracle import ref

pytestmark = pytest.mark.gpu

# K = 252, 1028, 512 and 1300
SHAPES = {"a": pv_inputs.ModelShape("vr_a", 1, 252, 4, 2, 128, 1028, 500, dtype="f32", seed=9301), "b": pv_inputs.ModelShape("vr_b", 1, 1028, 2, 1, 126, 1300, 333, dtype="f32", seed=9302)}


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("rows", [1, 2, 4, 5, 8, 9, 16, 17, 33, 64])
def test_rows_and_ragged_features(name, rows):
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    shape = SHAPES[name]
    gm, rm = gpu_model(shape, gains="perturbed", max_gamma=64), ref_model(shape, gains="perturbed")
    gc, rc = pv.Cache(gm, 128), ref.RefCache(rm, 128)
    toks = pv_inputs.uniform_tokens(87, 21 + rows, shape.vocab)
    gc.prefill(toks[:21]); rc.prefill(toks[:21])
    d = toks[21:].copy()
    d[0] = rc.pending
    n_r, t_r, pred_r, want = rc.verify(21, d, want_logits=True)
    n_g, t_g = gc.verify(21, d)
    assert np.abs(gc.debug_logits() - want).max() < 1e-4
    assert np.array_equal(gc.debug_pred(), pred_r) and (n_g, t_g) == (n_r, t_r)
