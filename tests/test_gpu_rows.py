"""Layer products above 64 rows (tiles of 96, 128 and 256 rows, K split across the grid): a layer against the oracle at
row counts around the tiles' edges, with output widths that leave the last column tile partly empty and contractions
shorter than the copy pipeline."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import make_ctx
from helpers import check_topk
from oracle import pie_oracle as O
from test_gpu_parity import compare_layer, small_model

pytestmark = pytest.mark.gpu


def mixed(T, n_decode=20):
    return [W.RequestSpec(1, 3 + 5 * i) for i in range(n_decode)] + [W.RequestSpec(T - n_decode, 19)]


@pytest.mark.parametrize("T", [65, 96, 97, 129, 192, 193, 289, 385])
def test_rows_around_the_96_row_tile(T):
    """hidden 320: five k steps, ten column blocks (two tiles, the second with two blocks); MLP 1088: seventeen k steps
    of the down projection, split, and 68 gate/up blocks (the last tile half empty)."""
    m = small_model(64, 8, 2, hidden=320, mlp=1088, vocab=512)
    w = W.build_workload("rows", m, mixed(T), n_kv_pages=200, seed=400 + T, std=0.02, resid_std=0.01)
    compare_layer(w, what=f"T={T} H320 I1088")


@pytest.mark.parametrize("T", [388, 511, 512])
def test_rows_around_the_128_row_tile(T):
    """64 column tiles: 128-row tiles fill the chip in one round where 96-row tiles need a second one (gate/up: two k
    steps, fewer than the copy pipeline is deep)."""
    m = small_model(64, 4, 2, hidden=128, mlp=8192, vocab=512)
    w = W.build_workload("rows128", m, mixed(T), n_kv_pages=200, seed=500 + T, std=0.02, resid_std=0.02 / 8)
    compare_layer(w, what=f"T={T} H128 I8192")


@pytest.mark.parametrize("rows,vocab", [(97, 1184), (129, 1184), (200, 2080), (300, 1184), (900, 352)])
def test_lm_head_with_any_number_of_tiles(rows, vocab):
    """Column tiles in numbers that are no multiple of the XCDs (37, 65 and 11 blocks of 32: 5, 9 and 2 tiles) by two and more
    row tiles: each XCD's range of tiles begins at a place of its own."""
    m = small_model(64, 4, 2, hidden=320, mlp=320, vocab=vocab)
    w = W.build_workload("head", m, [W.RequestSpec(1, 3)], n_kv_pages=4, seed=600 + rows, std=0.02, n_embeds=rows)
    ctx = make_ctx(w, max_dist_rows=rows, max_top_k=16)
    ids = np.random.default_rng(rows).permutation(rows).astype(np.int32)
    ctx.embed_write(ids, O.bf16_encode(np.random.default_rng(rows + 1).standard_normal((rows, m.hidden)).astype(np.float32)))
    emb = O.EmbedPool(rows, m.hidden)
    emb.write(ids, ctx.embed_read(ids))
    gi, gp = ctx.get_next_dist(ids, 16, 1.0)
    oi, op, z = O.get_next_dist(m, w.head, emb, ids, 16, 1.0, round_intermediates=True)
    check_topk(gi, gp, z, oi, op)
