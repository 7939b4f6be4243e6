"""GPU tests of cached steps whose lookup reads the first of the output weights ahead of the launch that streams them: vocabularies
whose blocks of 32 words do not divide evenly among the 256 workgroups, steps of few new histories (streamed) and of many (not),
one and two row blocks, each kernel that has a streaming form; against the oracle, tolerances as in test_gpu_cache.py.
"""
import numpy as np
import pytest

import oracle
import paper_2007_11794_amd as rn

from harness import CachedStepper, load_model
from test_gpu_cache import compare, draw_step, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V,H,max_rows,ids_of", [
    ("bf16", 70001, 320, 4500, (40, 30, 100, 4200)),     # staged; more ids than the small grouping takes in the last step
    ("bf16", 33001, 1020, 300, (33, 64, 90)),            # row streaming
    ("f32", 33000, 300, 200, (20, 32, 70)),              # two terms
    ("bf16", 70001, 256, 60, (60, 1)),                   # the streaming kernel itself
])
def test_steps_with_weights_read_ahead(dtype, V, H, max_rows, ids_of):
    rng = np.random.default_rng(V + H)
    K = 3
    model = small_model(rng, V, H, dtype, 0.05)
    m = load_model(model, dtype, max_rows)
    cache, ocache = rn.rnnlm_cache_create(m, 1000), oracle.Cache(H, 1000)
    st = CachedStepper(m, cache, max_rows, K)
    for step, ids in enumerate(ids_of):
        pool = np.arange(min(ids, 100), dtype=np.uint64) + np.uint64(50 * step)       # half of them known from the step before
        ids, prev, h_in, query, base = draw_step(rng, V, H, max(ids, max_rows - step) if ids < 100 else ids, K, pool)
        out = st.step(ids, prev, h_in, query, base)
        ref = oracle.step_cached(model, ocache, ids, prev, h_in, query, base_score=base)
        compare(out, ref, dtype, "%s V=%d H=%d step %d" % (dtype, V, H, step))
    assert cache.stats() == ocache.stats()
    assert m.last_error() == 0
    cache.close()
    m.close()
