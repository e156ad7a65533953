"""16-bit weights: output and down projections cut along K over workgroups (k_gemm_wide with K-slices, k_tile_finish behind it) against the oracle, on both sides of the lines from which they are
cut, and in a step that takes its buffers from the fixed array, with and without room for the slices' sums."""
import numpy as np
import pytest

import pv_inputs
from test_gpu_matrix import _check_against_oracle, pvlib  # noqa: F401

pytestmark = pytest.mark.gpu

S = pv_inputs.ModelShape
# 32 strips in 16 slices of 11 K-tiles and less (172 of them); 34 strips, a group of two at the end, in 16 slices (405 K-tiles); 128 strips in eight slices of 23 K-tiles and less (177)
SHAPES = [S("wcut_a", 1, 512, 8, 2, 64, 5504, 512, rope_base=500000.0, dtype="bf16", seed=7781), S("wcut_b", 1, 544, 8, 2, 64, 12960, 512, dtype="bf16", seed=7782),
          S("wcut_c", 1, 2048, 8, 2, 64, 5664, 512, dtype="bf16", seed=7783)]
BLOCKS = (9, 16, 8, 5, 1, 13, 17, 33, 64, 24)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda v: v.name)
def test_cut_projections_match_oracle(pvlib, shape):  # noqa: F811
    _check_against_oracle(pvlib, shape, 0, 64, 20, BLOCKS, 320)


def _cut(call):
    """K-slices' launches of k_gemm_wide (the last template argument 4) in a call."""
    import torch
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU, torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
    return sum("k_gemm_wide<" in e.name and e.name.split(">")[0].endswith(", 4") for e in p.events())


# d_model, K of the down projection -> {rows: cut projections of the layer}.  The output projection (K = 512) is cut from 17 rows on where the groups of four strips are a multiple of eight.
@pytest.mark.parametrize("d,k,cut", [(512, 256, {17: 1, 48: 1, 64: 1}), (512, 480, {17: 1, 33: 1, 64: 1}), (512, 512, {17: 2, 64: 2}),
                                     (512, 3328, {16: 0}), (512, 3520, {16: 1, 9: 1, 8: 0}), (512, 7040, {8: 0}), (512, 8192, {8: 1, 4: 0, 17: 2, 64: 2}), (512, 12800, {4: 0}), (512, 14336, {4: 1}),
                                     (512, 16384, {32: 2, 48: 2}), (512, 16416, {17: 1, 33: 1, 64: 1}), (640, 2048, {17: 0, 64: 0}), (4096, 8000, {16: 0}), (4096, 8576, {16: 1}), (4096, 4096, {32: 2}),
                                     (4096, 4128, {32: 1})])
def test_where_projections_are_cut(pvlib, d, k, cut):  # noqa: F811
    from gpu_helpers import gpu_model
    gm = gpu_model(S("wcut_line", 1, d, 8, 2, 64, k, 512, dtype="bf16", seed=7790), max_gamma=64)
    c = pvlib.Cache(gm, 192)
    c.use_graphs(False)
    c.prefill(pv_inputs.uniform_tokens(5, 5, 512))
    for rows, expected in cut.items():
        c.rollback(5)
        draft = pv_inputs.uniform_tokens(6, rows, 512)
        assert _cut(lambda: c.verify(5, draft)) == expected, rows


def test_cut_in_the_fixed_array(pvlib):  # noqa: F811
    """The step without allocations does the same; where the array has no room for the sums the projection stays whole, and steps that fitted before still do."""
    from gpu_helpers import gpu_model
    gm = gpu_model(SHAPES[0], max_gamma=16)
    prompt, draft = pv_inputs.uniform_tokens(7, 20, 512), pv_inputs.uniform_tokens(8, 12, 512)
    a = pvlib.Cache(gm, 96)
    a.prefill(prompt)
    draft[0] = a.pending
    want = a.verify(20, draft)

    def step(tokens, call=None):
        c = pvlib.Cache(gm, tokens)
        c.prefill(prompt)
        n = _cut(lambda: c.verify_async_static(20, draft)) if call else c.verify_async_static(20, draft)
        assert c.verify_wait() == want
        return c, n

    b, n = step(96, call=True)
    assert n == 1 and np.array_equal(a.export(), b.export())
    lo, hi = 96, 1 << 21                                        # the longest cache whose step fits
    with pytest.raises(Exception, match="fixed array"):
        step(hi)
    while hi - lo > 1024:
        mid = (lo + hi) // 2
        try:
            step(mid)
            lo = mid
        except Exception as e:
            assert "fixed array" in str(e)
            hi = mid
    c, n = step(lo, call=True)
    assert n == 0
    got, ref = c.export().astype(np.uint32) << 16, a.export().astype(np.uint32) << 16
    assert np.abs(got.view(np.float32) - ref.view(np.float32)).max() < 2e-2
