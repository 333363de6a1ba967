"""Calls that take an id list from the host pass it as kernel arguments up to 960 ids and through device memory beyond: Embed
writes and reads byte for byte, and distributions, around both argument sizes."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import make_ctx
from oracle import pie_oracle as O
from test_gpu_parity import small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("final_norm", [True, False])
def test_embeds_and_distributions_over_any_number_of_ids(final_norm):
    m = small_model(hidden=288, vocab=512)
    w = W.build_workload("ids", m, [W.RequestSpec(1, 3)], n_kv_pages=4, seed=5, std=0.05, n_embeds=1500)
    if not final_norm:
        w.head.g_final = None
    ctx = make_ctx(w, max_dist_rows=961, max_top_k=4)
    rng = np.random.default_rng(7)
    held = np.zeros((1500, m.hidden), np.uint16)
    everything = np.arange(1500, dtype=np.int32)
    ctx.embed_write(everything, held)
    for n in (1, 63, 64, 65, 959, 960, 961):
        ids = rng.permutation(1500)[:n].astype(np.int32)
        held[ids] = O.bf16_encode(rng.standard_normal((n, m.hidden)).astype(np.float32))
        ctx.embed_write(ids, held[ids])
        assert np.array_equal(ctx.embed_read(ids), held[ids]), n
        assert np.array_equal(ctx.embed_read(everything), held), n  # and nothing else was written
        gi, gp = ctx.get_next_dist(ids, 4, 1.0)
        emb = O.EmbedPool(1500, m.hidden)
        emb.write(ids, held[ids])
        oi, op, z = O.get_next_dist(m, w.head, emb, ids, 4, 1.0, round_intermediates=True)
        assert np.mean(gi == oi) > 0.99, n  # (nearly equal logits may change places)
        # (a normalised input near 4 that rounds the other way, 2^-6, moves a logit by up to 2^-6 x 0.2: two of them)
        np.testing.assert_allclose(gp, op, rtol=1e-2, err_msg=str(n))
