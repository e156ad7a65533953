"""What a step costs depends on the tokens that are cached, not on how many the cache has room for."""
import time

import numpy as np
import pytest

import pv_inputs

pytestmark = pytest.mark.gpu

# Little but attention: 8 layers of 32 query heads on narrow projections
HEADS = pv_inputs.ModelShape("room", 8, 256, 32, 8, 128, 256, 256, dtype="bf16", seed=7701)


def test_the_merge_of_the_chunks_reads_what_was_launched():
    """600 cached tokens, 64 rows, recorded and plain steps: with room for 32768 tokens the merge has 8 and 6 chunks to look at and not 256.  Reading
    outputs for all 256 took 543 us a step instead of 460; now 459 and 460.  The bound lies in the middle of the two ratios, 1.18 and 1.00."""
    import torch
    import paper_2505_01572_amd as pv
    from gpu_helpers import gpu_model
    gm = gpu_model(HEADS, max_gamma=64)
    prompt, draft = pv_inputs.uniform_tokens(3, 600, HEADS.vocab), pv_inputs.uniform_tokens(4, 64, HEADS.vocab)
    caches = [pv.Cache(gm, n) for n in (700, 32768)]
    for c in caches:
        c.prefill(prompt)
        c.set_pending(int(draft[0] + 1) % HEADS.vocab)         # nothing is accepted: the step can be repeated
    logits = []
    for graphs in (True, False):
        best = [1e9, 1e9]
        for c in caches:
            c.use_graphs(graphs)
            c.verify(600, draft)
            logits.append(c.debug_logits())
        for _ in range(8):
            for i, c in enumerate(caches):
                torch.cuda.synchronize()
                t = time.perf_counter()
                for _ in range(20):
                    c.verify(600, draft)
                best[i] = min(best[i], time.perf_counter() - t)
        print(f"graphs {graphs}: {best[0] / 20 * 1e6:.1f} us and {best[1] / 20 * 1e6:.1f} us")
        assert best[1] < 1.09 * best[0]
    for lg in logits[1:]:
        assert np.array_equal(lg, logits[0])
