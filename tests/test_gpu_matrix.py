"""GPU parity of the matrix-core (MFMA) path on small bf16 shapes that still span several
tiles, ragged K splits and both operand packings (rows <= 8 and 9..16).

Oracle: fp64 arithmetic on the same bf16 weights, K/V rounded to bf16 on store (the cache's
storage type).  Bar for bf16 storage: max |dlogit| <= 3e-2 x RMS(logits) per row; the split
hi/lo activations should do ~100x better, which is asserted too so a precision regression shows.
"""
import numpy as np
import pytest

import pv_inputs
from oracle import ref
from helpers import ref_model

pytestmark = pytest.mark.gpu

MAT_A = pv_inputs.ModelShape("mat_a", 3, 128, 8, 2, 32, 352, 512, rope_base=500000.0, dtype="bf16", seed=5151)
MAT_B = pv_inputs.ModelShape("mat_b", 2, 1024, 8, 2, 128, 4128, 2000, rope_base=500000.0, dtype="bf16", seed=5252)
MAT_C = pv_inputs.ModelShape("mat_c", 2, 512, 8, 8, 64, 1376, 1008, dtype="bf16", seed=5353)   # MHA, hd 64
# larger K (multiples of 256): 16-wave K split with several tiles per wave, long ragged down-projection slice
FUSE_A = pv_inputs.ModelShape("fuse_a", 2, 512, 8, 2, 64, 1280, 1008, rope_base=500000.0, dtype="bf16", seed=5454)
FUSE_B = pv_inputs.ModelShape("fuse_b", 2, 1024, 8, 2, 128, 8448, 2000, rope_base=500000.0, dtype="bf16", seed=5555)
# K = d_model = 65 tiles: the waves walk their batches several deep and a ragged tile is left over; 512 gate/up strips and
# 512 vocabulary strips put two strips in a workgroup, 130 down-projection strips one
DEEP_A = pv_inputs.ModelShape("deep_a", 2, 2080, 8, 2, 128, 4096, 8192, rope_base=500000.0, dtype="bf16", seed=5656)


@pytest.fixture(scope="module")
def pvlib():
    import torch
    assert torch.cuda.is_available()
    import paper_2505_01572_amd as pv
    return pv


def _rel_err(pvlib, lg_g, lg_r):
    from gpu_helpers import logit_scale
    return (np.abs(lg_g - lg_r) / logit_scale(lg_r)).max()


CASES = [(MAT_A, 0), (MAT_B, 0), (MAT_C, 0), (FUSE_A, 0), (FUSE_B, 2), (DEEP_A, 0)]


def _check_against_oracle(pvlib, shape, path, max_gamma, prompt_len, gammas, cache_tokens):
    from gpu_helpers import gpu_model, top2_margin
    gm = gpu_model(shape, gains="perturbed", kernel_path=path, max_gamma=max_gamma)
    rm = ref_model(shape, gains="perturbed")
    prompt = pv_inputs.uniform_tokens(61, prompt_len, shape.vocab)
    gc, rc = pvlib.Cache(gm, cache_tokens), ref.RefCache(rm, cache_tokens, ref.KV_BF16)
    gc.prefill(prompt)                      # chunks of max_gamma rows and a ragged last one
    last = rc.prefill(prompt)
    assert _rel_err(pvlib, gc.debug_logits()[-1:], last[None]) < 2e-3
    assert gc.state() == (prompt_len, rc.pending)
    worst = 0.0
    for step, gamma in enumerate(gammas):
        T = len(rc)
        d = pv_inputs.uniform_tokens(62 + step, gamma, shape.vocab)
        if rc.pending >= 0:                  # (unknown after a rollback: the first draft token is then trusted)
            d[0] = rc.pending
        n_r, t_r, pred_r, lg_r = rc.verify(T, d, want_logits=True)
        n_g, t_g = gc.verify(T, d)
        lg_g = gc.debug_logits()
        err = _rel_err(pvlib, lg_g, lg_r)
        worst = max(worst, err)
        assert err < 3e-2, f"gamma {gamma}: {err}"
        safe = top2_margin(lg_r) > 4 * np.abs(lg_g - lg_r).max()
        assert np.array_equal(gc.debug_pred()[safe], pred_r[safe])
        if safe[: max(n_r, 1)].all():
            assert (n_g, t_g) == (n_r, t_r) and gc.state() == (len(rc), rc.pending)
        else:                                # a near-tie decided the step: follow the oracle
            gc.rollback(T); rc.rollback(T)
    assert worst < 2e-3, worst
    ge = pv_inputs.bf16_bits_to_f32(gc.export()).astype(np.float64)
    re_ = rc.export()
    print(f"{shape.name}: worst rel logit err {worst:.2e}, KV 1-ulp flips {np.mean(ge != re_):.4f}")
    assert ge.shape == re_.shape and np.mean(ge != re_) < 0.02     # 1-ulp bf16 flips at rounding boundaries only
    assert np.abs(ge - re_).max() <= 2.0 ** -7 * np.abs(re_).max()


@pytest.mark.parametrize("shape,path", CASES, ids=lambda v: v.name if hasattr(v, "name") else f"path{v}")
def test_matrix_path_matches_oracle(pvlib, shape, path):
    _check_against_oracle(pvlib, shape, path, 16, 37, (8, 13, 1, 5, 16, 3), 96)   # prefill chunks of 16, 16, 5 rows


@pytest.mark.parametrize("name", ["mat_a", "mat_b", "fuse_b", "q4_b"])
def test_packed_rows_match_oracle(pvlib, name):
    """Every number of rows that is packed into one operand tile; the down projections of mat_b (129 K-tiles, 64 strips) and
    fuse_b (264) run as half strips."""
    shape = {"mat_a": MAT_A, "mat_b": MAT_B, "fuse_b": FUSE_B, "q4_b": Q4_B}[name]
    _check_against_oracle(pvlib, shape, 0, 16, 21, (2, 7, 4, 6, 1, 3, 5, 8), 96)


def test_chunks_beyond_four_per_lane(pvlib):
    """33000 cached positions: 259 chunks of 128 keys (gamma 8) take the merge's general path, 130 of 256 keys (gamma 4) do not.  Against the vector path, which
    has no chunks."""
    from gpu_helpers import gpu_model
    T0 = 33000
    prompt = pv_inputs.uniform_tokens(65, T0, LONG_A.vocab)
    caches = [pvlib.Cache(gpu_model(LONG_A, gains="perturbed", kernel_path=p, max_gamma=16), T0 + 64) for p in (pvlib.PATH_AUTO, pvlib.PATH_VECTOR)]
    for c in caches:
        c.prefill(prompt)
    for step, gamma in enumerate((8, 4)):
        d = pv_inputs.uniform_tokens(66 + step, gamma, LONG_A.vocab)
        lg = []
        for c in caches:
            c.verify(T0, d)
            lg.append(c.debug_logits())
            c.rollback(T0)
        assert _rel_err(pvlib, lg[0], lg[1]) < 2e-3, f"gamma {gamma}"


# Output projections that merge the attention's chunks: K = 2048 as half strips and as whole ones (130), 4096 features with one row; 3..8 chunks of 256 keys
MERGE = [pv_inputs.ModelShape("merge_h", 1, 1024, 32, 8, 64, 352, 512, dtype="bf16", seed=5901),
         pv_inputs.ModelShape("merge_w", 1, 2080, 16, 2, 128, 352, 512, dtype="bf16", seed=5902),
         pv_inputs.ModelShape("merge_k", 1, 512, 32, 4, 128, 352, 512, dtype="bf16", seed=5903)]


@pytest.mark.parametrize("shape", MERGE, ids=lambda v: v.name)
@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("prefix", [509, 700, 1022, 1500, 2046])
def test_merged_chunks_match_oracle(pvlib, shape, graphs, prefix):
    """One and two rows around the edges of the chunks; recorded steps cover chunks beyond the keys (of an earlier, longer prefix), plain ones do not."""
    from gpu_helpers import gpu_model
    gm, rm = gpu_model(shape, gains="perturbed", max_gamma=16), ref_model(shape, gains="perturbed")
    gc, rc = pvlib.Cache(gm, 2112), ref.RefCache(rm, 2112, ref.KV_BF16)
    gc.use_graphs(graphs)
    prompt = pv_inputs.uniform_tokens(81, 2048, shape.vocab)
    gc.prefill(prompt)
    gc.verify(2048, prompt[:1])
    gc.rollback(prefix)
    rc.prefill(prompt[:prefix])
    for step, gamma in enumerate((1, 2, 1, 3)):
        T = len(rc)
        d = pv_inputs.uniform_tokens(82 + step, gamma, shape.vocab)
        _, _, _, lg_r = rc.verify(T, d, want_logits=True)
        n, _ = gc.verify(T, d)
        assert _rel_err(pvlib, gc.debug_logits(), lg_r) < 2e-3, f"gamma {gamma} at {T}"
        gc.rollback(T); rc.rollback(T)


# The same with chunks of 128 keys: more than 16 query rows per kv head, in one group of 32 (16 heads and two rows, 32 heads and one) or two (32 heads and two)
MERGE_128 = [pv_inputs.ModelShape("merge_g", 1, 1024, 32, 2, 64, 352, 512, dtype="bf16", seed=5904),
             pv_inputs.ModelShape("merge_u", 1, 1024, 32, 1, 64, 352, 512, dtype="bf16", seed=5905)]


@pytest.mark.parametrize("shape", MERGE_128, ids=lambda v: v.name)
@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("prefix", [256, 383, 509, 700, 1021])
def test_merged_chunks_of_128_keys_match_oracle(pvlib, shape, graphs, prefix):
    """256 .. 510 keys are three or four chunks, merged by the output projection for one row and for two; up to 1023 five to eight, for one."""
    test_merged_chunks_match_oracle(pvlib, shape, graphs, prefix)


def test_chunks_of_128_keys_are_merged_by_the_output_projection(pvlib):
    """Which kernel that test is about: the last template argument is the most chunks it merges."""
    import re
    import torch
    from gpu_helpers import gpu_model
    for shape, merges in zip(MERGE_128, ({(2, 300): 4, (2, 600): 0, (1, 300): 0, (1, 600): 4}, {(1, 300): 4, (2, 300): 4, (1, 600): 8, (2, 600): 0})):
        gc = pvlib.Cache(gpu_model(shape, max_gamma=16), 1100)
        gc.use_graphs(False)
        gc.prefill(pv_inputs.uniform_tokens(83, 1000, shape.vocab))
        for (rows, prefix), most in sorted(merges.items(), key=lambda v: -v[0][1]):
            gc.rollback(prefix)
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU, torch.profiler.ProfilerActivity.CUDA]) as p:
                gc.verify(prefix, pv_inputs.uniform_tokens(84, rows, shape.vocab))
            found = [re.match(r"(?:void )?k_gemm<([^>]*)>", e.name) for e in p.events()]
            got = [int(f[1].split(",")[7]) for f in found if f and f[1].split(",")[3].strip() == "1"]
            assert sorted(got) == sorted([0, most]), (shape.name, rows, prefix, got)


def test_wide_blocks_match_oracle(pvlib, wide_shape):
    """Blocks of 17..64 rows (two and four 16-row column tiles per weight pass; with 4-bit weights one
    weight pass per column tile), next to narrow ones on the same cache; the prompt is prefilled in
    64-row chunks plus a ragged rest."""
    _check_against_oracle(pvlib, wide_shape, 0, 64, 100, (32, 17, 64, 8, 40, 1, 33), 320)


# A workgroup per CU with 3, 6, 7, 4 and 7 strips (vocabularies of 705, 1500, 1601, 1009 and 1537 strips), ragged in the strips, with 17 K-tiles (not a multiple
# of the waves) or 129 (9..16 rows take that kernel from 128 on); in the first shape the QKV and gate/up projections (720 and 708 strips) as well.
WIDE = [pv_inputs.ModelShape("wide_3", 1, 544, 60, 60, 64, 5664, 705 * 16, dtype="bf16", seed=5801),
        pv_inputs.ModelShape("wide_6", 1, 544, 8, 2, 32, 352, 1500 * 16, dtype="bf16", seed=5802),
        pv_inputs.ModelShape("wide_7", 1, 544, 8, 2, 32, 352, 1601 * 16, dtype="bf16", seed=5803),
        pv_inputs.ModelShape("wide_k", 1, 4128, 8, 2, 32, 352, 1009 * 16, dtype="bf16", seed=5804),
        pv_inputs.ModelShape("wide_p", 1, 4128, 8, 2, 32, 352, 1537 * 16, dtype="bf16", seed=5805)]


@pytest.mark.parametrize("shape", WIDE, ids=lambda v: v.name)
def test_one_workgroup_per_cu_matches_oracle(pvlib, shape):
    """Every number of column tiles at its first and last row count (33..48 rows: three); up to 8 rows from 1025 strips and 128 K-tiles on."""
    _check_against_oracle(pvlib, shape, 0, 64, 20, (17, 32, 33, 48, 49, 64, 9, 16, 8, 1, 5), 320)


# Packed rows at the lower end of one workgroup per CU (1024 strips: two a workgroup) and inside (1376: six, ragged; K = 4128)
WIDE_PACKED = [pv_inputs.ModelShape("wide_p4", 1, 4128, 8, 2, 32, 352, 1024 * 16, dtype="bf16", seed=5806),
               pv_inputs.ModelShape("wide_p6", 1, 4128, 8, 2, 32, 352, 1376 * 16, dtype="bf16", seed=5807)]


@pytest.mark.parametrize("shape", WIDE_PACKED, ids=lambda v: v.name)
def test_packed_rows_with_one_workgroup_per_cu_match_oracle(pvlib, shape):
    _check_against_oracle(pvlib, shape, 0, 16, 20, (8, 1, 2, 3, 4, 5, 6, 7), 320)


LONG_A = pv_inputs.ModelShape("long_a", 1, 128, 8, 2, 32, 352, 512, rope_base=500000.0, dtype="bf16", seed=5757)


def test_long_prefix_many_attention_chunks(pvlib):
    """8300 cached positions: with 32 query rows per kv head (gamma 8, group 4) attention makes 65
    chunks of 128 keys, more than the lanes of a wave; with 16 rows (gamma 4) it makes 33 chunks of 256 keys."""
    from gpu_helpers import gpu_model
    gm = gpu_model(LONG_A, gains="perturbed", kernel_path=0, max_gamma=64)
    rm = ref_model(LONG_A, gains="perturbed")
    T0 = 8300
    prompt = pv_inputs.uniform_tokens(63, T0, LONG_A.vocab)
    gc, rc = pvlib.Cache(gm, T0 + 64), ref.RefCache(rm, T0 + 64, ref.KV_BF16)
    gc.prefill(prompt)
    last = rc.prefill(prompt)
    assert _rel_err(pvlib, gc.debug_logits()[-1:], last[None]) < 2e-3
    for step, gamma in enumerate((8, 4, 1, 16)):
        T = len(rc)
        d = pv_inputs.uniform_tokens(64 + step, gamma, LONG_A.vocab)
        if rc.pending >= 0:
            d[0] = rc.pending
        n_r, t_r, pred_r, lg_r = rc.verify(T, d, want_logits=True)
        gc.verify(T, d)
        assert _rel_err(pvlib, gc.debug_logits(), lg_r) < 2e-3, f"gamma {gamma}"
        gc.rollback(T); rc.rollback(T)          # every block on the same 8300-token prefix


def test_matrix_and_vector_paths_agree(pvlib):
    from gpu_helpers import gpu_model
    ma = gpu_model(MAT_A, gains="perturbed")
    va = gpu_model(MAT_A, gains="perturbed", kernel_path=pvlib.PATH_VECTOR)
    prompt = pv_inputs.uniform_tokens(71, 20, MAT_A.vocab)
    a, b = pvlib.Cache(ma, 64), pvlib.Cache(va, 64)
    a.prefill(prompt); b.prefill(prompt)
    assert a.state() == b.state()
    d = pv_inputs.uniform_tokens(72, 8, MAT_A.vocab); d[0] = a.pending
    ra, rb = a.verify(20, d), b.verify(20, d)
    la, lb = a.debug_logits(), b.debug_logits()
    assert np.abs(la - lb).max() < 2e-3 * np.sqrt((lb ** 2).mean())
    assert ra == rb


def test_matrix_rollback_and_paging(pvlib):
    from gpu_helpers import gpu_model
    gm = gpu_model(MAT_A, gains="perturbed")
    a, b = pvlib.Cache(gm, 96), pvlib.Cache(gm, 96)
    b.set_page_table(np.array([4, 2, 0, 5, 1, 3], dtype=np.int32))
    toks = pv_inputs.uniform_tokens(81, 60, MAT_A.vocab)
    for c in (a, b):
        c.prefill(toks[:29])
    before, pend = a.export(), a.pending
    d = toks[29:40].copy(); d[0] = pend
    ra, rb = a.verify(29, d), b.verify(29, d)
    lg = a.debug_logits()
    assert ra == rb and np.array_equal(lg, b.debug_logits()) and lg.shape == (11, MAT_A.vocab)
    assert np.array_equal(a.export(), b.export())       # (export reuses the logits buffer)
    a.rollback(29)
    assert np.array_equal(a.export(), before)
    a.set_pending(pend)
    assert a.verify(29, d) == ra and np.array_equal(a.debug_logits(), lg)   # bit-identical rerun


def test_matrix_block_equals_sequential(pvlib):
    from gpu_helpers import gpu_model
    gm = gpu_model(MAT_C, gains="perturbed")
    toks = pv_inputs.uniform_tokens(91, 30, MAT_C.vocab)
    a, b = pvlib.Cache(gm, 64), pvlib.Cache(gm, 64)
    a.prefill(toks[:19]); b.prefill(toks[:19])
    a.set_pending(-1)
    a.verify(19, toks[19:27])
    blk = a.debug_logits()
    seq = []
    for t in toks[19:27]:
        b.rollback(len(b))
        n, _ = b.verify(len(b), [t]); assert n == 1
        seq.append(b.debug_logits()[0])
    scale = np.sqrt((blk ** 2).mean())
    assert np.abs(blk - np.stack(seq)).max() < 1e-3 * scale


def test_graph_replay_equals_plain_launches(pvlib):
    """The step recorded as a HIP graph must give, on every replay, exactly what the plain launch
    sequence gives: same accepted length, next token, predictions, logits bit for bit and the
    same K/V.  Each row count is replayed several times, with unrelated eager GPU work and
    synchronisations between the replays; both matrix (bf16) and vector (fp32) paths."""
    import torch
    from gpu_helpers import gpu_model
    tiny = pv_inputs.CONFIGS["tiny"]
    for shape in (FUSE_A, tiny):
        gm = gpu_model(shape, gains="perturbed")
        cg, cp = pvlib.Cache(gm, 256), pvlib.Cache(gm, 256)
        cp.use_graphs(False)
        prompt = pv_inputs.uniform_tokens(71, 41, shape.vocab)
        cg.prefill(prompt); cp.prefill(prompt)          # 16-row chunks: the prefill graphs replay too
        assert cg.state() == cp.state()
        junk = torch.zeros(1 << 20, device="cuda")
        for step, gamma in enumerate((8, 8, 3, 8, 16, 3, 1, 16, 8, 1, 3, 8)):
            T, pending = cp.state()
            d = pv_inputs.uniform_tokens(720 + step, gamma, shape.vocab)
            if step % 3 != 2 and pending >= 0:
                d[0] = pending
            r_p = cp.verify(T, d)
            junk.add_(1.0); s = float(junk.sum().item())   # eager kernels (a multi-block reduction among them) + sync
            assert s == (step + 1) * junk.numel()
            r_g = cg.verify(T, d)
            assert r_g == r_p, (shape.name, step, gamma)
            assert np.array_equal(cg.debug_pred(), cp.debug_pred())
            assert np.array_equal(cg.debug_logits(), cp.debug_logits()), (shape.name, step, gamma)
            assert cg.state() == cp.state()
            if step == 5:                                  # an external rollback between replays
                cg.rollback(T); cp.rollback(T)
        assert np.array_equal(cg.export(), cp.export())


# ---- 4-bit weights (codes + bf16 group scales): the projections and the LM head ----

Q4_A = pv_inputs.ModelShape("q4_a", 3, 128, 8, 2, 32, 384, 512, rope_base=500000.0, dtype="bf16", seed=7171, weight_bits=4)
Q4_B = pv_inputs.ModelShape("q4_b", 2, 1024, 8, 2, 128, 4224, 2000, rope_base=500000.0, dtype="bf16", seed=7272, weight_bits=4)
Q4_C = pv_inputs.ModelShape("q4_c", 2, 512, 8, 8, 64, 1408, 1008, dtype="bf16", seed=7373, weight_bits=4)   # MHA, hd 64
# K = d_model = 17 batches (odd shares per wave); 512 gate/up strips: two per workgroup, 1024 vocabulary strips: four
Q4_D = pv_inputs.ModelShape("q4_d", 2, 2176, 8, 2, 128, 4096, 16384, rope_base=500000.0, dtype="bf16", seed=7474, weight_bits=4)


@pytest.fixture(params=["mat_a", "mat_c", "fuse_a", "q4_a", "q4_c"])
def wide_shape(request):
    return {"mat_a": MAT_A, "mat_c": MAT_C, "fuse_a": FUSE_A, "q4_a": Q4_A, "q4_c": Q4_C}[request.param]


@pytest.mark.parametrize("shape", [Q4_A, Q4_B, Q4_C, Q4_D], ids=lambda v: v.name)
def test_q4_weights_match_oracle(pvlib, shape):
    """The oracle runs the same decoder on the dequantised weights (code - 8) * scale; the library
    streams codes and scales and dequantises inside the matrix-core GEMMs."""
    _check_against_oracle(pvlib, shape, 0, 16, 37, (8, 13, 1, 5, 16, 3), 96)


# Two, three (one round of workgroups and two), four and seven strips a workgroup (vocabularies of 300, 705, 1300 and 1009 strips, 1616 strips of gate/up), ragged
# in the strips; 1, 5 or 9 batches along K for eight waves; 404 K-tiles and 3700 strips, where 9..16 rows go back to shared tiles.
Q4_STRIPS = [pv_inputs.ModelShape("q4_s2", 1, 1152, 8, 2, 64, 384, 300 * 16, dtype="bf16", seed=7581, weight_bits=4),
             pv_inputs.ModelShape("q4_s3", 1, 640, 8, 2, 64, 12928, 705 * 16, dtype="bf16", seed=7582, weight_bits=4),
             pv_inputs.ModelShape("q4_s3b", 1, 128, 8, 2, 32, 384, 1300 * 16, dtype="bf16", seed=7583, weight_bits=4),
             pv_inputs.ModelShape("q4_s4", 1, 1152, 8, 2, 64, 384, 1009 * 16, dtype="bf16", seed=7584, weight_bits=4),
             pv_inputs.ModelShape("q4_sx", 1, 128, 8, 2, 32, 384, 3700 * 16, dtype="bf16", seed=7585, weight_bits=4)]


@pytest.mark.parametrize("shape", Q4_STRIPS, ids=lambda v: v.name)
def test_q4_strips_of_a_workgroup_match_oracle(pvlib, shape):
    _check_against_oracle(pvlib, shape, 0, 16, 20, (8, 16, 1, 4, 5, 9), 96)


def test_q4_model_is_smaller_and_rejects_plain_loads(pvlib):
    import paper_2505_01572_amd as pv
    m4 = pv.Model(Q4_B, max_gamma=16)
    m16 = pv.Model(Q4_B.replace(weight_bits=16), max_gamma=16)
    assert m4.weight_bytes < 0.45 * m16.weight_bytes
    rows = np.zeros((16, Q4_B.d_model), dtype=np.uint16)
    with pytest.raises(pv.PVError):
        m4.load_weights("wq", 0, 0, rows)                   # a 4-bit matrix does not take bf16 rows
    with pytest.raises(pv.PVError):
        m16.load_weights_q4("wq", 0, 0, np.zeros((16, Q4_B.d_model // 2), np.uint8), np.zeros((16, Q4_B.d_model // 32), np.uint16))
    pv.Model(Q4_B, max_gamma=64)                            # wide blocks: one weight pass per 16-row column tile
