"""Products above 64 rows: a layer against the oracle at row counts around the edges of the 96- and 128-row tiles, with
output widths that leave the last column tile partly empty and contractions shorter than the copy pipeline; each form the
products are cut into (tiles of 96, 128 and 256 rows, K whole or split, whole rounds and a remainder), with the partial
sums handed to the rotary step, the second norm and the next layer; LM heads."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import assert_mlp_stages, gpu_forward, make_ctx, product_forms
from helpers import check_topk
from oracle import pie_oracle as O
from test_gpu_model import compare_deep
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


@pytest.mark.parametrize("T,shape,forms", [
    # split gate/up; every partial sum at up to 256 rows
    (130, dict(head_dim=64, n_q=16, n_kv=4, hidden=1024, mlp=1024), {"qkv": (96, 4, 0), "o": (96, 4, 0), "gateup": (96, 4, 0)}),
    # partial sums of QKV and O handed on above 256 rows
    (300, dict(head_dim=64, n_q=16, n_kv=4, hidden=1024, mlp=2048), {"qkv": (96, 4, 0), "o": (96, 4, 0), "down": (96, 8, 0)}),
    # ... and where a rotary thread walks eight heads (1024 tokens and more)
    (1060, dict(head_dim=64, n_q=16, n_kv=4, hidden=2048, mlp=1024), {"qkv": (96, 2, 0)}),
    # 128-row tiles, split
    (1000, dict(head_dim=128, n_q=16, n_kv=4, hidden=2048, mlp=1024), {"o": (128, 3, 0), "gateup": (128, 3, 0)}),
])
def test_split_products(T, shape, forms):
    m = small_model(**shape, vocab=512)
    got = product_forms(m, T)
    assert {k: got[k] for k in forms} == forms
    w = W.build_workload("split", m, mixed(T), n_kv_pages=T // 16 + 240, seed=700 + T, std=0.02, resid_std=0.01)
    compare_layer(w, what=f"T={T} H{m.hidden} I{m.mlp_dim}")


def test_256_row_tiles_split_and_whole_rounds_with_a_remainder():
    """Nine rows of 256-row tiles with K in three parts (down), and eight of them with twelve rows left over (gate/up)."""
    m, T = small_model(64, 16, 4, hidden=2048, mlp=8192, vocab=512), 2060
    got = product_forms(m, T)
    assert got["down"] == (256, 3, 0) and got["gateup"] == (256, 1, 2048)
    w = W.build_workload("tall", m, mixed(T), n_kv_pages=400, seed=710, std=0.02, resid_std=0.005)
    ctx = make_ctx(w, with_head=False)
    _, stored, y_bits = gpu_forward(ctx, w)
    assert len(stored) == T
    from paper_2510_24051_amd import TAP_ACT, TAP_RESID
    pick = np.unique(np.concatenate([np.arange(0, T, 17), [255, 256, 511, 512, 2047, 2048, 2059]]))  # rows of every tile
    assert_mlp_stages(w, ctx.read_tap(TAP_RESID, T)[pick], ctx.read_tap(TAP_ACT, T)[pick], y_bits[pick], pick, f"T={T}")


@pytest.mark.parametrize("T", [100, 290])
def test_down_projection_partials_carried_to_the_next_layer(T):
    """Two layers through forward_all: the first one's down projection leaves its parts to the second one's first norm."""
    m = small_model(64, 16, 4, hidden=1024, mlp=2048, vocab=512)
    m.n_layers = 2
    assert product_forms(m, T)["down"] == (96, 8, 0)
    dw = W.build_deep_workload("carried", m, mixed(T), n_kv_pages=T // 16 + 240, seed=720 + T, std=0.02, resid_std=0.005)
    compare_deep(dw, f"carried T={T}")
