"""Projections over more features than 32-bit buffer offsets reach: blocks of up to 16 rows run them in kernels with 64-bit addresses.  Compared with the same rows at the
head of a block of 24, which shares its activation tiles through LDS and has 64-bit addresses throughout."""
import ctypes

import numpy as np
import pytest

import pv_inputs

pytestmark = pytest.mark.gpu


class _Staging:
    """The library with a staging buffer that holds 16 rows of such a matrix (what pv_model_bytes reports is the least)."""

    def __init__(self, real, nbytes):
        self._real, self._nbytes = real, nbytes

    def __getattr__(self, name):
        return getattr(self._real, name)

    def pv_model_bytes(self, cfg, weights, staging):
        rc = self._real.pv_model_bytes(cfg, weights, staging)
        staging._obj.value = max(staging._obj.value, self._nbytes)
        return rc


@pytest.mark.parametrize("bits", [16, 4])
@pytest.mark.parametrize("ktiles", [1 << 19, (1 << 19) + 4, (1 << 20) + 4], ids=["last_within", "first_past", "past_2_25"])
def test_a_down_projection_past_the_offsets(monkeypatch, ktiles, bits):
    import torch
    import paper_2505_01572_amd as pv
    from gpu_helpers import logit_scale
    F, d = 32 * ktiles, 32 if bits == 16 else 128
    shape = pv_inputs.ModelShape("far", 1, d, d // 32, 1, 32, F, 64, dtype="bf16", weight_bits=bits)
    real = pv.lib()
    monkeypatch.setattr(pv.binding, "lib", lambda: _Staging(real, 16 * F * 2 + 512))
    m = pv.Model(shape, max_gamma=64, prompt_rows=0)
    # a pool of draws whose length is odd: what lies a power of two away is something else
    rng = np.random.default_rng(9)
    n = 16_000_003
    if bits == 16:
        pool = torch.from_numpy(rng.standard_normal(n, dtype=np.float32) * 0.05).to(torch.bfloat16).view(torch.uint16).numpy()
    else:
        codes, scales = rng.integers(0, 256, n, dtype=np.uint8), rng.integers(0x3C00, 0x3C80, n, dtype=np.uint16)      # scales of 2^-7 .. 2^-6
    for kind, layer in pv_inputs.iter_tensors(shape):
        dims = pv_inputs.tensor_shape(shape, kind)
        rows, cols = (1, dims[0]) if len(dims) == 1 else dims
        if rows == 1:
            m.load_weights(kind, layer, 0, np.full((1, cols), 0x3F80, np.uint16))
            continue
        step = 16 if cols == F else min(rows, 1 << 18)
        for r0 in range(0, rows, step):
            k = min(step, rows - r0)
            if bits == 4 and kind in pv_inputs.Q4_KINDS:
                m.load_weights_q4(kind, layer, r0, np.resize(np.roll(codes, r0 + 1), (k, cols // 2)), np.resize(np.roll(scales, r0 + 1), (k, cols // 32)))
            else:
                src = pool if bits == 16 else np.full(1, 0x3D00, np.uint16) + (rng.integers(0, 2, 4099, dtype=np.uint16) << 15)
                m.load_weights(kind, layer, r0, np.resize(np.roll(src, r0 + 1), (k, cols)))
    c = pv.Cache(m, 64)
    c.prefill(pv_inputs.uniform_tokens(1, 3, 64))
    block = pv_inputs.uniform_tokens(2, 24, 64)
    c.set_pending(int(block[0] + 1) % 64)                      # nothing is accepted
    c.verify(3, block)
    want = c.debug_logits()
    assert np.isfinite(want).all()
    for rows in (1, 5, 8, 9, 16):
        c.verify(3, block[:rows])
        got = c.debug_logits()
        assert (np.abs(got - want[:rows]) / logit_scale(want[:rows])).max() < 2e-3, rows
    c.close(); m.close()
