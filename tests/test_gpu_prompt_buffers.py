"""The buffers of long prompts: one set behind a model's weights, none in its caches; fewer rows or none at all; whatever they
hold; prompts of several caches at once."""
import functools
import threading

import numpy as np
import pytest

import pv_inputs

pytestmark = pytest.mark.gpu

SHAPES = {"bf16": pv_inputs.ModelShape("pb_16", 2, 512, 8, 2, 64, 1408, 1008, rope_base=500000.0, seed=7501),
          "q4": pv_inputs.ModelShape("pb_q4", 2, 512, 8, 2, 64, 1408, 1008, rope_base=500000.0, seed=7502, weight_bits=4)}


def _left_behind(c):
    return c.state(), c.debug_logits(), c.debug_pred(), c.export()


def _same(a, b):
    return a[0] == b[0] and all(np.array_equal(x, y) for x, y in zip(a[1:], b[1:]))


def test_a_cache_holds_no_prompt_buffers():
    """Between 64 and 2048 tokens a workspace grows by the page table and the attention partials (256 keys each) only."""
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    shape = SHAPES["bf16"]
    gm = gpu_model(shape, max_gamma=64)
    small, large = pv.Cache(gm, 64), pv.Cache(gm, 2048)
    units = 64 * (shape.n_q_heads // shape.n_kv_heads) // 32 + 16 * 2
    partials = 16 * units * shape.n_kv_heads * 32 * (shape.head_dim + 2) * 4
    assert large.ws.numel() - small.ws.numel() < 2 * partials + 4 * 2048 + 4096


@pytest.mark.parametrize("name", SHAPES)
@pytest.mark.parametrize("rows", [0, 64, 65, 192, 320])
def test_fewer_rows_a_pass(monkeypatch, name, rows):
    """Down to none: then prompts go in as blocks of 64, bit for bit."""
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model, logit_scale
    monkeypatch.setattr(pv, "Model", functools.partial(pv.Model, prompt_rows=rows))
    shape = SHAPES[name]
    gm = gpu_model(shape, gains="perturbed")
    toks = pv_inputs.uniform_tokens(75, 450, shape.vocab)
    a, b = pv.Cache(gm, 500), pv.Cache(gm, 500)
    a.prefill(toks)
    for i in range(0, 450, 64):
        b.prefill(toks[i:i + 64])
    a, b = _left_behind(a), _left_behind(b)
    if rows <= 64:
        assert _same(a, b)
    la, lb = a[1], b[1]
    assert la.shape == lb.shape and (np.abs(la - lb) / logit_scale(lb)).max() < 2e-3


@pytest.mark.parametrize("name", SHAPES)
def test_whatever_the_buffers_hold(name):
    """NaN bit patterns everywhere before the prompt (a pass of 300 rows leaves the last row tile and rectangle partly unused)."""
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    shape = SHAPES[name]
    gm = gpu_model(shape, gains="perturbed")
    toks = pv_inputs.uniform_tokens(76, 300, shape.vocab)
    got = []
    for fill in (0, 255):
        gm.arena[gm.weight_bytes:].fill_(fill)
        c = pv.Cache(gm, 320)
        c.prefill(toks)
        got.append(_left_behind(c))
    assert np.isfinite(got[0][1]).all() and _same(*got)


def test_prompts_of_several_caches_at_once():
    """Four threads with a stream and a cache each: as one after the other, bit for bit."""
    import torch
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    shape = SHAPES["bf16"]
    gm = gpu_model(shape, gains="perturbed")
    prompts = [pv_inputs.uniform_tokens(80 + i, n, shape.vocab) for i, n in enumerate((2300, 700, 130, 2100))]
    want = []
    for p in prompts:
        c = pv.Cache(gm, 2400)
        c.prefill(p)
        want.append(_left_behind(c))
    for _ in range(3):
        caches = [pv.Cache(gm, 2400) for _ in prompts]
        streams = [torch.cuda.Stream() for _ in prompts]
        torch.cuda.synchronize()
        threads = [threading.Thread(target=c.prefill, args=(p, s)) for c, p, s in zip(caches, prompts, streams)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert all(_same(_left_behind(c), w) for c, w in zip(caches, want))


@pytest.mark.parametrize("n", [60, 300, 2300])
def test_a_prompt_and_the_first_step_create_no_stream(n):
    """The stream on which steps are recorded comes with the cache: creating it takes as long as a fifth of a step, and stops kernels that run."""
    import torch
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    shape = SHAPES["bf16"]
    gm = gpu_model(shape)
    c = pv.Cache(gm, n + 16)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU, torch.profiler.ProfilerActivity.CUDA]) as p:
        c.prefill(pv_inputs.uniform_tokens(81, n, shape.vocab))
        c.verify(n, [c.pending, 1, 2, 3])
    calls = {e.name for e in p.events()}
    assert "hipGraphLaunch" in calls and not any(x.startswith("hipStreamCreate") for x in calls), calls
