"""Long prompts (more than 64 tokens in one prefill call) against the CPU oracle and against the same prompt put in as
64-token pieces: lengths at the edges of the row rectangles (16, 64, 128, 256) and of a pass (2048), head dimensions and
group sizes, a prefix already in the cache, shuffled pages, ragged strip counts, K cut into slices."""
import numpy as np
import pytest

import pv_inputs
from helpers import ref_model
from oracle import ref

pytestmark = pytest.mark.gpu

S = pv_inputs.ModelShape
SHAPES = {
    "gqa64": S("pr_gqa64", 2, 512, 8, 2, 64, 1408, 1008, rope_base=500000.0, seed=7101),          # 88 gate/up strips x 2, ragged rectangles
    "mha128": S("pr_mha128", 2, 256, 3, 3, 128, 736, 512, seed=7102),                             # no sharing of K/V heads, K of 8, 12 and 23 tiles
    "odd32": S("pr_odd32", 2, 160, 15, 5, 32, 96, 512, seed=7103),                                # three heads to a kv head; K of 5, 15 and 3 tiles
    "deep": S("pr_deep", 1, 1024, 8, 1, 128, 8448, 2000, rope_base=500000.0, seed=7104),          # long K: cut into slices; eight heads to a kv head
    "q4": S("pr_q4", 2, 512, 8, 2, 64, 1408, 1008, rope_base=500000.0, seed=7105, weight_bits=4),
    "q4_deep": S("pr_q4_deep", 1, 1024, 8, 2, 128, 8448, 2000, rope_base=500000.0, seed=7106, weight_bits=4),
}
CASES = [("gqa64", 0, 65, 64), ("gqa64", 3, 80, 16), ("deep", 0, 128, 16), ("gqa64", 0, 129, 64), ("gqa64", 0, 257, 16), ("gqa64", 37, 300, 16), ("gqa64", 128, 192, 64), ("mha128", 5, 400, 16), ("mha128", 0, 145, 16),
         ("odd32", 0, 520, 16), ("odd32", 70, 131, 32), ("deep", 0, 260, 16), ("deep", 3, 600, 128), ("gqa64", 0, 2048 + 70, 16), ("gqa64", 9, 2048 + 200, 16),
         ("q4", 0, 129, 16), ("q4", 37, 300, 16), ("q4_deep", 0, 260, 16), ("q4_deep", 3, 600, 16)]


@pytest.mark.parametrize("name,before,n,page", CASES)
def test_long_prompt(name, before, n, page):
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model, logit_scale
    shape = SHAPES[name].replace(page_tokens=page)
    gm = gpu_model(shape, gains="perturbed")
    toks = pv_inputs.uniform_tokens(71, before + n, shape.vocab)
    room = before + n + 24
    pages = -(-room // page)
    a, b = pv.Cache(gm, room), pv.Cache(gm, room)
    a.set_page_table(np.random.default_rng(3).permutation(pages))
    if before:
        a.prefill(toks[:before])
    a.prefill(toks[before:])
    if before:
        b.prefill(toks[:before])
    for i in range(before, before + n, 64):
        b.prefill(toks[i:min(i + 64, before + n)])
    lg, lb = a.debug_logits(), b.debug_logits()
    # rows, logits and prediction of the last block of 64, whatever the prompt went in as
    assert lg.shape == lb.shape == ((n - 1) % 64 + 1, shape.vocab)
    scale = logit_scale(lb)
    assert (np.abs(lg - lb) / scale).max() < 2e-3
    margin = np.sort(lb, axis=1)
    safe = margin[:, -1] - margin[:, -2] > 4 * np.abs(lg - lb).max()
    assert np.array_equal(a.debug_pred()[safe], b.debug_pred()[safe])
    assert len(a) == len(b) == before + n
    if safe[-1]:
        assert a.state() == b.state()
    ka, kb = (pv_inputs.bf16_bits_to_f32(c.export()).astype(np.float64) for c in (a, b))
    assert np.mean(ka != kb) < 0.02 and np.abs(ka - kb).max() <= 2.0 ** -7 * np.abs(kb).max()     # one bf16 step at rounding boundaries
    d = pv_inputs.uniform_tokens(72, 8, shape.vocab)
    d[0] = a.pending
    a.verify(before + n, d)
    lv = a.debug_logits()
    if before + n <= 620:
        rm = ref_model(shape, gains="perturbed")
        rc = ref.RefCache(rm, room, ref.KV_BF16)
        last = rc.prefill(toks)
        assert (np.abs(lg[-1] - last) / logit_scale(last)).max() < 2e-3
        _, _, _, want = rc.verify(before + n, d, want_logits=True)
        assert (np.abs(lv - want) / logit_scale(want)).max() < 2e-3
    else:
        b.set_pending(int(d[0]))
        b.verify(before + n, d)
        assert (np.abs(lv - b.debug_logits()) / logit_scale(lv)).max() < 2e-3


def test_non_finite_prompt_commits_all_but_the_last_block():
    """Weights that make every logit NaN: the last 64-token block is not committed, as with short prompts."""
    import paper_2505_01572_amd as pv
    shape = SHAPES["gqa64"]
    from gpu_helpers import gpu_model
    gm = gpu_model(shape)
    bad = np.full((1, shape.d_model), 0x7FC0, dtype=np.uint16)
    gm.load_weights("final_norm", 0, 0, bad)
    c = pv.Cache(gm, 400)
    with pytest.raises(pv.PVError) as e:
        c.prefill(pv_inputs.uniform_tokens(5, 300, shape.vocab))
    assert e.value.status == -6
    assert c.state() == (256, -1)


def test_rollback_and_readmit_after_a_long_prompt():
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    shape = SHAPES["gqa64"]
    gm = gpu_model(shape, gains="perturbed")
    toks = pv_inputs.uniform_tokens(73, 400, shape.vocab)
    a, b = pv.Cache(gm, 480), pv.Cache(gm, 480)
    a.prefill(toks[:300])
    a.rollback(150)
    a.prefill(toks[150:])
    b.prefill(toks[:150]); b.prefill(toks[150:])
    assert a.state() == b.state() and np.array_equal(a.export(), b.export())
    # the block on record is the prompt's last one of 64: all of it is committed, so there is nothing but its end to go to
    c = pv.Cache(gm, 480)
    for n in (300, 100):
        c.prefill(toks[:n])
        for bad in (len(c) - 1, len(c) + 1):
            with pytest.raises(pv.PVError) as e:
                c.readmit(bad)
            assert e.value.status == -3
        c.readmit(len(c), pending=9)
        assert c.state()[1] == 9
    c.rollback(350)
    with pytest.raises(pv.PVError) as e:
        c.readmit(400)
    assert e.value.status == -2 and c.state() == (350, -1)
    # a last block that was not committed can be re-admitted, wholly or in part: its keys and values are there
    good = pv_inputs.fill_tensor(shape, "final_norm", -1, gains="perturbed").reshape(1, -1)
    for before, n, to in ((0, 300, 300), (0, 300, 257), (7, 2048 + 100, 7 + 2048 + 64 + 30)):
        full = pv_inputs.uniform_tokens(74, before + n, shape.vocab)
        c, d = pv.Cache(gm, before + n + 8), pv.Cache(gm, before + n + 8)
        gm.load_weights("final_norm", 0, 0, np.full((1, shape.d_model), 0x7FC0, dtype=np.uint16))
        if before:
            with pytest.raises(pv.PVError):
                c.prefill(full[:before])
            c.readmit(before)
        with pytest.raises(pv.PVError):
            c.prefill(full[before:])
        kept = before + n - ((n - 1) % 64 + 1)
        assert c.state() == (kept, -1)
        for bad in (kept - 1, before + n + 1):
            with pytest.raises(pv.PVError) as e:
                c.readmit(bad)
            assert e.value.status == -3
        c.readmit(to, pending=5)
        assert c.state() == (to, 5)
        gm.load_weights("final_norm", 0, 0, good)
        if before:
            d.prefill(full[:before])
        d.prefill(full[before:])
        d.rollback(to); d.set_pending(5)
        assert c.verify(to, [5, 1, 2]) == d.verify(to, [5, 1, 2]) and np.array_equal(c.debug_logits(), d.debug_logits())


@pytest.mark.parametrize("bits", [0x3580, 0x4600, 0x8000, 0xBC00], ids=["small", "large", "minus_zero", "negative"])
def test_scales_at_the_ends(bits):
    """4-bit weights go into long prompts as 16-bit floats unless some scale of the model does not fit that form
    (0x3580 = 2^-20, 0x4600 = 2^13; -0 and negative scales fit): either way as with the blocks of 64 tokens, which use the bf16 scales as they are."""
    import paper_2505_01572_amd as pv
    from gpu_helpers import logit_scale, paired_models
    shape = SHAPES["q4"]
    gm, _ = paired_models(shape)
    arr = pv_inputs.fill_tensor(shape, "wo", 0).reshape(pv_inputs.tensor_shape(shape, "wo"))
    codes, scales = pv_inputs.quantize_q4(arr)
    scales[5, 3] = bits
    gm.load_weights_q4("wo", 0, 0, codes, scales)
    toks = pv_inputs.uniform_tokens(74, 200, shape.vocab)
    a, b = pv.Cache(gm, 256), pv.Cache(gm, 256)
    a.prefill(toks)
    for i in range(0, 200, 64):
        b.prefill(toks[i:i + 64])
    la, lb = a.debug_logits(), b.debug_logits()
    assert np.isfinite(la).all() and (np.abs(la - lb) / logit_scale(lb)).max() < 2e-3


def test_large_activations_of_a_4bit_model():
    """An FFN gain of 2^20: operands of 2^20 and (SwiGLU) some 2^38, whose rows are scaled before they become 16-bit floats.  (Larger
    gains would overflow the sums of squares in fp32 on any path.)"""
    import paper_2505_01572_amd as pv
    from gpu_helpers import logit_scale, paired_models
    shape = SHAPES["q4"]
    gm, _ = paired_models(shape)
    gm.load_weights("ffn_norm", 0, 0, np.full((1, shape.d_model), 0x4980, dtype=np.uint16))
    toks = pv_inputs.uniform_tokens(75, 200, shape.vocab)
    a, b = pv.Cache(gm, 256), pv.Cache(gm, 256)
    a.prefill(toks)
    for i in range(0, 200, 64):
        b.prefill(toks[i:i + 64])
    la, lb = a.debug_logits(), b.debug_logits()
    assert np.isfinite(lb).all() and np.abs(lb).max() > 0 and (np.abs(la - lb) / logit_scale(lb)).max() < 2e-3


@pytest.mark.parametrize("name,before,n,page", [("gqa64", 1000, 5000, 16), ("mha128", 700, 4400, 64), ("q4", 300, 4500, 16)])
def test_several_passes(name, before, n, page):
    test_long_prompt(name, before, n, page)


@pytest.mark.parametrize("heads,kv_heads,head_dim", [(2, 2, 128), (8, 2, 64), (4, 1, 128)])
def test_attention_error_does_not_grow_with_the_context(heads, kv_heads, head_dim):
    """A prompt of one repeated token: all values are equal, so attention's exact output, and with one layer every row's
    logits, are those of the single token whatever the length.  What 12000 keys add in rounding errors stays within 1.4 times what
    300 add (rms over 40 or more rows; one accumulator over all keys: 1.5 to 2.2 times)."""
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model, logit_scale
    shape = S("pr_same", 1, 256, heads, kv_heads, head_dim, 352, 512, rope_base=500000.0, seed=7401, page_tokens=64)
    wo = pv_inputs.fill_tensor(shape, "wo", 0).reshape(pv_inputs.tensor_shape(shape, "wo"))
    large = {("wo", 0): (wo + np.uint16(4 << 7)).astype(np.uint16)}                # times 16: attention's output dominates the residual
    gm = gpu_model(shape, gains="perturbed", overrides=large)
    want = ref.RefCache(ref_model(shape, gains="perturbed", overrides=large), 8, ref.KV_BF16).prefill(np.array([7], dtype=np.int32))
    one = pv.Cache(gm, 8)
    one.prefill([7])
    base = one.debug_logits()
    rms = {}
    for n in (300, 12000):
        c = pv.Cache(gm, n)
        c.prefill(np.full(n, 7, dtype=np.int32))
        lg = c.debug_logits()
        assert len(lg) >= 32 and np.sqrt((((lg - want) / logit_scale(want)) ** 2).mean()) < 4e-6
        rms[n] = np.sqrt((((lg - base) / logit_scale(want)) ** 2).mean())
    assert rms[12000] < 1.4 * rms[300], rms


def _first_values(d, n):
    """A one-layer model, n tokens, and its first layer's values in 64 bits, rounded: no attention in them yet."""
    import torch
    from gpu_helpers import gpu_model
    shape = S("pr_exact_%d" % d, 1, d, 16, 16, 128, 96, 4096, seed=7402, page_tokens=64)
    toks = pv_inputs.uniform_tokens(76, n, shape.vocab)
    w = {k: torch.from_numpy(pv_inputs.bf16_bits_to_f32(pv_inputs.fill_tensor(shape, k, l, gains="perturbed").reshape(pv_inputs.tensor_shape(shape, k))).astype(np.float64))
         for k, l in (("embed", -1), ("attn_norm", 0), ("wv", 0))}
    x = w["embed"][torch.from_numpy(toks.astype(np.int64))]
    want = (x * torch.rsqrt((x * x).mean(1, keepdim=True) + shape.rms_eps) * w["attn_norm"]) @ w["wv"].t()
    return gpu_model(shape, gains="perturbed"), toks, want.to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("d", [1024, 2048, 2080])
def test_values_of_a_long_prompt_are_as_exact_as_those_of_short_blocks(d):
    """As many of a first layer's values are not the rounded 64-bit result as with blocks of 64 tokens, give or take
    a tenth.  (Some 1400 of 8 million at d = 2048, a standard deviation of 4 % for the ratio; accumulators over 16 K-tiles, twice
    the blocks' 8, had 23 % more.)"""
    import paper_2505_01572_amd as pv
    n = 4000
    gm, toks, want = _first_values(d, n)
    a, b = pv.Cache(gm, n), pv.Cache(gm, n)
    a.prefill(toks)
    for i in range(0, n, 64):
        b.prefill(toks[i:i + 64])
    off = [np.count_nonzero(c.export()[0, 1] != want) for c in (a, b)]
    assert off[1] < 4e-4 * want.size and off[0] < 1.1 * off[1], off


@pytest.mark.parametrize("d,rows", [(3072, 24), (3072, 64), (4096, 24), (4096, 48)])
def test_values_of_wide_blocks_against_64_bits(d, rows):
    """Blocks of 17 to 64 rows: 1.8 to 1.9 in 10000 first-layer values are not the rounded 64-bit result (of 8 million: a standard deviation of 3 %),
    as with K-slices of 8 tiles; accumulators over 16 K-tiles had 2.2 to 2.4."""
    import paper_2505_01572_amd as pv
    n = 4000
    gm, toks, want = _first_values(d, n)
    c = pv.Cache(gm, n)
    for i in range(0, n, rows):
        c.prefill(toks[i:i + rows])
    assert np.count_nonzero(c.export()[0, 1] != want) < 2.1e-4 * want.size


def _reload(gm, rm, shape, kind, layer, bits):
    """The tensor again with one scale replaced (None: none), on both sides."""
    codes, scales = pv_inputs.quantize_q4(pv_inputs.fill_tensor(shape, kind, layer).reshape(pv_inputs.tensor_shape(shape, kind)))
    if bits is not None:
        scales[5, 3] = bits
    rm.set_tensor(kind, layer, ref.dequant_q4(codes, scales))
    step = gm.chunk_rows(2 * codes.shape[1])
    for r0 in range(0, codes.shape[0], step):
        gm.load_weights_q4(kind, max(layer, 0), r0, codes[r0:r0 + step], scales[r0:r0 + step])


@pytest.mark.parametrize("kind,layer,scaled", [("lm_head", -1, set()), ("wk", 1, {"k_pre_gemm_q4<4, 0>"}), ("wd", 0, {"k_pre_gemm_q4<4, 1>"}), ("wu", 1, {"k_pre_gemm_q4<4, 2>"})])
def test_a_scale_decides_for_its_own_matrices(kind, layer, scaled):
    """One scale of 2^-20: the GEMM with that matrix takes the kernel that scales its products, once in the two layers, all others keep
    the weights as 16-bit floats (the vocabulary projection has no part in it); and so does that one when the tensor is loaded again without it."""
    import torch
    import paper_2505_01572_amd as pv
    from gpu_helpers import paired_models
    shape = SHAPES["q4"]
    gm, rm = paired_models(shape)
    toks = pv_inputs.uniform_tokens(77, 200, shape.vocab)
    for bits, expected in ((0x3580, scaled), (None, set())):
        _reload(gm, rm, shape, kind, layer, bits)
        c = pv.Cache(gm, 256)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU, torch.profiler.ProfilerActivity.CUDA]) as p:
            c.prefill(toks)
        names = [e.name.replace("void ", "").split("(")[0] for e in p.events()]
        got = [n for n in names if n.startswith("k_pre_gemm_q4")]
        assert set(got) == expected and len(got) == len(expected)
        assert len([n for n in names if n.startswith("k_pre_gemm_h4")]) == 8 - len(expected)


Q4_LONG = S("pr_q4_long", 1, 1408, 8, 2, 64, 1664, 1008, rope_base=500000.0, seed=7107, weight_bits=4)


@pytest.mark.parametrize("before,n,bits", [(40, 2048, 0x3580), (0, 2048 + 300, 0x4600), (40, 2048, None)])
def test_long_prompts_of_4bit_models_with_an_uncut_k(before, n, bits):
    """2048 rows and 208 gate/up strips: 208 rectangles, so K (44 K-tiles, no multiple of the 8 of an accumulator) is not cut; several row
    rectangles on every XCD.  With a scale that does not fit 16-bit floats in each matrix (2^-20 or 2^13), and without."""
    import paper_2505_01572_amd as pv
    from gpu_helpers import logit_scale, paired_models
    shape = Q4_LONG
    gm, rm = paired_models(shape)
    for kind in ("wq", "wo", "wg", "wd") if bits else ():
        _reload(gm, rm, shape, kind, 0, bits)
    toks = pv_inputs.uniform_tokens(78, before + n, shape.vocab)
    a, b = pv.Cache(gm, before + n + 8), pv.Cache(gm, before + n + 8)
    rc = ref.RefCache(rm, before + n + 8, ref.KV_BF16)
    for c in (a, b):
        if before:
            c.prefill(toks[:before])
    a.prefill(toks[before:])
    for i in range(before, before + n, 64):
        b.prefill(toks[i:min(i + 64, before + n)])
    last, la, lb = rc.prefill(toks), a.debug_logits(), b.debug_logits()
    assert (np.abs(la[-1] - last) / logit_scale(last)).max() < 2e-3 and (np.abs(la - lb) / logit_scale(lb)).max() < 2e-3
    ka, kb = (pv_inputs.bf16_bits_to_f32(c.export()).astype(np.float64) for c in (a, b))
    assert np.mean(ka != kb) < 0.02 and np.abs(ka - kb).max() <= 2.0 ** -7 * np.abs(kb).max()


@pytest.mark.parametrize("spread", [8, 20, 30])
def test_rows_of_a_4bit_model_with_a_wide_spread(spread):
    """Norm gains of 2^-spread to 1 side by side: a row's elements differ by as much before they become 16-bit floats, down to below the
    2^-22 of the largest from which on those hold fewer bits.  As exact as blocks of 64 tokens, against the oracle."""
    import paper_2505_01572_amd as pv
    from gpu_helpers import logit_scale, paired_models
    shape = SHAPES["q4"]
    gm, rm = paired_models(shape)
    rng = np.random.default_rng(spread)
    for kind in ("attn_norm", "ffn_norm"):
        for layer in range(shape.n_layers):
            gain = ((127 - rng.integers(0, spread + 1, (1, shape.d_model))) << 7).astype(np.uint16)
            gm.load_weights(kind, layer, 0, gain)
            rm.set_tensor(kind, layer, gain.reshape(-1))
    toks = pv_inputs.uniform_tokens(79, 200, shape.vocab)
    a, b, rc = pv.Cache(gm, 256), pv.Cache(gm, 256), ref.RefCache(rm, 256, ref.KV_BF16)
    a.prefill(toks)
    for i in range(0, 200, 64):
        b.prefill(toks[i:i + 64])
    last, la, lb = rc.prefill(toks), a.debug_logits(), b.debug_logits()
    ea, eb = (np.sqrt((((x[-1] - last) / logit_scale(last)) ** 2).mean()) for x in (la, lb))
    assert (np.abs(la - lb) / logit_scale(lb)).max() < 2e-3 and ea < 2 * eb + 1e-5, (ea, eb)
    ka, kb = (pv_inputs.bf16_bits_to_f32(c.export()).astype(np.float64) for c in (a, b))
    assert np.mean(ka != kb) < 0.02 and np.abs(ka - kb).max() <= 2.0 ** -7 * np.abs(kb).max()
