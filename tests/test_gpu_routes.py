"""Which kernel a projection takes, at both sides of the lines that the launches draw: a line in the wrong place is a block that takes up to twice its time
and fails no other test.  (Where the lines lie, and the measurements on both sides, stands at the launches.)  The block's logits are compared with those of
the same rows in blocks of eight, which run other kernels."""
import re

import numpy as np
import pytest

import pv_inputs

pytestmark = pytest.mark.gpu

SWIGLU, LMHEAD = 2, 3          # the epilogue's number among a kernel's template arguments
EPI_AT = {"k_gemm": 3, "k_gemm_wide": 3, "k_gemm_tile": 2, "k_gemm_q4": 2, "k_gemm_tile_q4": 1}


def _model(k, strips, bits=16, ffn=256):
    """One layer of width k with a vocabulary of `strips` strips (gate/up: ffn / 8); every matrix is windows of one pool of normal draws."""
    import torch
    import paper_2505_01572_amd as pv
    shape = pv_inputs.ModelShape("route", 1, k, k // 128, 1, 128, ffn, 16 * strips, weight_bits=bits)
    m = pv.Model(shape, max_gamma=64, prompt_rows=0)
    rng = np.random.default_rng(77)
    pool = torch.from_numpy(rng.standard_normal(1 << 22, dtype=np.float32) * 0.02).to(torch.bfloat16).view(torch.uint16).numpy()
    for kind, layer in pv_inputs.iter_tensors(shape):
        dims = pv_inputs.tensor_shape(shape, kind)
        rows, cols = (1, dims[0]) if len(dims) == 1 else dims
        if rows == 1:
            m.load_weights(kind, layer, 0, np.full((1, cols), 0x3F80, np.uint16))
            continue
        step = max(16, min(m.chunk_rows(cols), pool.size // cols // 16 * 16))
        for r0 in range(0, rows, step):
            n = min(step, rows - r0)
            at = int(rng.integers(0, max(1, pool.size - n * cols)))
            w = np.resize(pool[at:at + n * cols], (n, cols))
            if bits == 4 and kind in pv_inputs.Q4_KINDS:
                m.load_weights_q4(kind, layer, r0, *pv_inputs.quantize_q4(w))
            else:
                m.load_weights(kind, layer, r0, w)
    return m


def _head_kernel(call, epi=LMHEAD):
    """Name and template arguments of the kernel that multiplies with the vocabulary (of another projection: epi)."""
    import torch
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU, torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
    found = set()
    for e in p.events():
        hit = re.match(r"(?:void )?(k_gemm\w*)<([^>]*)>", e.name)
        if hit and hit[1] in EPI_AT:
            args = [int(v) if v.strip().isdigit() else v.strip() for v in hit[2].split(",")]
            if args[EPI_AT[hit[1]]] == epi:
                found.add((hit[1], *args))
    assert len(found) == 1, found
    return found.pop()


def _check(model, rows, logits=True, epi=LMHEAD):
    import paper_2505_01572_amd as pv
    from gpu_helpers import logit_scale
    v = model.shape.vocab
    prompt, block = pv_inputs.uniform_tokens(5, 5, v), pv_inputs.uniform_tokens(6, rows, v)
    a, b = pv.Cache(model, 96), pv.Cache(model, 96)
    a.use_graphs(False)
    for c in (a, b):
        c.prefill(prompt)
    name = _head_kernel(lambda: a.verify(5, block), epi)
    if logits:
        got, want = a.debug_logits(), []
        for r0 in range(0, rows, 8):
            b.prefill(block[r0:r0 + 8])
            want.append(b.debug_logits())
        want = np.concatenate(want)
        assert (np.abs(got - want) / logit_scale(want)).max() < 2e-3
    a.close(); b.close()
    return name


# K, strips -> {rows: takes k_gemm_wide}
WIDE_LINES = [
    (1024, 704, {32: True, 48: True, 64: True}), (1024, 700, {32: False, 64: False}),
    (1024, 1792, {32: True, 48: True, 64: True}), (1024, 2000, {32: False, 48: False, 64: False}),
    (1024, 2560, {32: True, 48: True, 64: True}), (1024, 3584, {32: True, 48: False, 64: False}),
    (1024, 4096, {32: False, 64: False}), (1024, 5120, {32: True, 48: False, 64: False}), (1024, 8016, {32: False, 48: False, 64: False}),
    (5120, 1024, {32: True, 64: True}), (5248, 1024, {32: False, 64: False}),
    (5120, 3584, {48: True}), (6656, 1792, {64: True}), (6784, 1792, {48: True, 64: False}),
    (4096, 704, {16: True}), (3968, 704, {16: False}),
]


@pytest.mark.parametrize("k,strips,expected", WIDE_LINES, ids=lambda v: str(v) if isinstance(v, int) else "")
def test_one_workgroup_per_cu_where_it_is_the_faster_one(k, strips, expected):
    m = _model(k, strips)
    for rows, wide in expected.items():
        name = _check(m, rows)
        assert (name[0] == "k_gemm_wide") == wide, (rows, name)
        if name[0] == "k_gemm_tile":
            assert name[1] == (rows + 15) // 16, name
    m.close()


# up to 8 rows: K, strips -> {rows: strips a workgroup, negative: of k_gemm_wide}
PACKED_LINES = [
    (4096, 1023, {1: 2, 8: 2}), (4096, 1024, {1: 2, 8: 2}), (4096, 1025, {1: -6, 8: -6}), (3968, 1088, {1: 1, 8: 1}), (4096, 1793, {1: 2, 8: 2}),
    (4096, 1199, {4: -6}), (4096, 1200, {4: 1, 5: -6}), (4608, 1280, {4: 1, 5: -6}), (4736, 1280, {1: -6}),
    (4096, 1350, {1: -6}), (4096, 1376, {1: 2, 4: 2, 5: -6, 8: -6}), (4096, 1439, {1: 2, 8: 2}), (4224, 1376, {1: -6}), (4224, 1440, {1: 2, 4: 2, 5: -6}),
    (5120, 1480, {8: -6}), (5120, 1488, {8: 2}), (7168, 1536, {1: 2, 8: 2}), (7296, 1536, {1: -6, 8: -6}),
    (4096, 1537, {1: -7, 8: -7}), (4096, 1679, {1: -7}), (4096, 1792, {1: 1, 5: -7, 8: -7}), (4736, 1792, {1: -7, 8: -7}),
]


@pytest.mark.parametrize("k,strips,expected", PACKED_LINES, ids=lambda v: str(v) if isinstance(v, int) else "")
def test_packed_rows_with_one_workgroup_per_cu(k, strips, expected):
    m = _model(k, strips)
    for rows, each in expected.items():
        name = _check(m, rows, logits=False)                   # (the same rows in blocks of eight would be the same kernel: the oracle tests have these)
        assert (name[0], name[3]) == ("k_gemm_wide" if each < 0 else "k_gemm", abs(each)), (rows, name)
    m.close()


# up to 8 rows, two strips a workgroup: K -> batches a wave keeps in flight
@pytest.mark.parametrize("k,depth", [(2048, 3), (3968, 3), (4096, 2), (5120, 2)])
def test_depth_of_two_packed_strips(k, depth):
    m = _model(k, 1024)
    for rows in (1, 8):
        name = _check(m, rows, logits=False)
        assert name[:7] == ("k_gemm", 1, 1, 2, LMHEAD, 8, depth), (rows, name)
    m.close()


# up to 8 rows, gate/up in 3 1/2 strips a workgroup: K -> {rows: strips a workgroup (4: the half ones), negative: of k_gemm_wide}
@pytest.mark.parametrize("k,expected", [(4096, {4: 1, 5: -7, 8: -7}), (4608, {4: 1, 5: 4, 8: 4}), (4736, {1: 4, 8: 4}), (7168, {1: 4, 8: 4}), (7296, {1: -7, 8: -7})])
def test_packed_gate_up_of_half_strips(k, expected):
    m = _model(k, 32, ffn=1792 * 8)
    for rows, each in expected.items():
        name = _check(m, rows, logits=False, epi=SWIGLU)
        assert (name[0], name[3]) == ("k_gemm_wide" if each < 0 else "k_gemm", abs(each)), (rows, name)
    m.close()


# 4-bit weights, up to 4 rows: K, strips -> waves of a workgroup
@pytest.mark.parametrize("k,strips,waves", [(512, 200, 8), (1920, 256, 8), (2048, 256, 16), (512, 512, 8), (1920, 300, 8), (2048, 512, 16), (2048, 513, 8)])
def test_sixteen_waves_where_each_has_a_batch(k, strips, waves):
    m = _model(k, strips, bits=4)
    for rows in (1, 4):
        name = _check(m, rows)
        assert name[0] == "k_gemm_q4" and name[4] == waves, (rows, name)
    assert _check(m, 5)[4] == 8
    m.close()


# 4-bit weights, 9..16 rows: K, strips -> strips a workgroup of k_gemm_q4, 0 where the tiles are shared
@pytest.mark.parametrize("k,strips,each", [(12800, 64, 1), (12928, 64, 0), (512, 1376, 3), (8192, 1100, 3), (8320, 1100, 0), (5376, 2304, 3), (5504, 2304, 0),
                                           (4096, 3300, 4), (4224, 3300, 0), (2048, 3584, 4), (512, 3584, 3), (512, 3585, 0)])
def test_unshared_tiles_of_4bit_blocks_of_9_to_16_rows(k, strips, each):
    m = _model(k, strips, bits=4)
    for rows in (9, 16):
        name = _check(m, rows)
        assert name[:3] == (("k_gemm_q4", 2, each) if each else ("k_gemm_tile_q4", 1, LMHEAD)), (rows, name)
    m.close()


# 4-bit weights, up to 8 rows: K, strips -> {rows: strips a workgroup}
@pytest.mark.parametrize("k,strips,each", [(2048, 1376, {1: 3, 7: 3, 8: 7}), (1920, 1376, {8: 3}), (2048, 1024, {1: 4, 8: 4}), (2048, 1025, {1: 3, 8: 7}), (512, 2000, {2: 4, 8: 4}),
                                           (2048, 3600, {1: 3, 8: 4}), (512, 8016, {1: 4, 8: 4})])
def test_strips_of_a_workgroup_by_the_rows(k, strips, each):
    m = _model(k, strips, bits=4)
    for rows, s in each.items():
        assert _check(m, rows)[2] == s, rows
    m.close()
