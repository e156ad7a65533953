"""4-bit weights, up to 16 rows: the down projection cut along K over workgroups (k_gemm_q4 with K-slices, k_tile_finish behind it) against the oracle, and
on both sides of the line from which it is cut."""
import pytest

import pv_inputs
from test_gpu_matrix import _check_against_oracle, pvlib  # noqa: F401

pytestmark = pytest.mark.gpu

S = pv_inputs.ModelShape
# 32 strips in 5 slices of 9 batches and less (43 of them); 64 strips in 13 of 9 (111); 40 strips, ten groups, in 12 of 9 (101)
SHAPES = [S("cut_a", 1, 512, 8, 2, 64, 5504, 512, rope_base=500000.0, dtype="bf16", seed=7681, weight_bits=4), S("cut_b", 1, 1024, 8, 2, 128, 14208, 512, dtype="bf16", seed=7682, weight_bits=4),
          S("cut_c", 1, 640, 8, 2, 64, 12928, 512, dtype="bf16", seed=7683, weight_bits=4)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda v: v.name)
def test_cut_down_projection_matches_oracle(pvlib, shape):  # noqa: F811
    _check_against_oracle(pvlib, shape, 0, 16, 20, (9, 16, 8, 5, 4, 1, 13), 96)


# d_model, K of the down projection -> {rows: whether it is cut}.  (operand bytes a CU does not read: 280 kB, 340 kB with other than a multiple of eight groups of four strips; a slice per 1024
# features at most)
@pytest.mark.parametrize("d,k,cut", [(512, 5376, {16: False}), (512, 5504, {16: True, 9: True, 8: False}), (512, 9728, {8: False, 16: True}), (512, 9856, {8: True, 7: False}), (640, 6272, {9: False}),
                                     (640, 6400, {9: True}), (512, 16512, {4: False}), (512, 16640, {4: True, 1: True})])
def test_where_the_down_projection_is_cut(pvlib, d, k, cut):  # noqa: F811
    import torch
    from gpu_helpers import gpu_model
    gm = gpu_model(S("cut_line", 1, d, 8, 2, 64, k, 512, dtype="bf16", seed=7690, weight_bits=4))
    c = pvlib.Cache(gm, 96)
    c.use_graphs(False)
    c.prefill(pv_inputs.uniform_tokens(5, 5, 512))
    for rows, expected in cut.items():
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU, torch.profiler.ProfilerActivity.CUDA]) as p:
            c.verify(len(c), pv_inputs.uniform_tokens(6, rows, 512))
        assert any("k_tile_finish" in e.name for e in p.events()) == expected, rows
