"""Layers of 1 to 32 tokens, whose products take in the norms, the rotary step and the epilogues: rows around the edges, both
head sizes, every row length, contractions that divide unevenly over the waves, column tiles in one and in several rounds, prompts
beside decode requests, several layers (wide residual in, wide residual out), pages of 32 tokens."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import make_ctx
from helpers import check_topk
from oracle import pie_oracle as O
from paper_2510_24051_amd import TAP_LOGITS
from test_gpu_adapter import compare as compare_adapters
from test_gpu_model import compare_deep
from test_gpu_parity import compare_layer, small_model

pytestmark = pytest.mark.gpu

# 2048 and 4096 wide: everything is taken in; 8192: q, k, v of the input Embeds; 96: nothing
SHAPES = [
    dict(head_dim=64, n_q=8, n_kv=2, hidden=2048, mlp=96),
    dict(head_dim=128, n_q=8, n_kv=2, hidden=4096, mlp=4128),
    dict(head_dim=64, n_q=12, n_kv=3, hidden=4096, mlp=8224),
    dict(head_dim=64, n_q=4, n_kv=2, hidden=96, mlp=160),
    dict(head_dim=128, n_q=4, n_kv=4, hidden=8192, mlp=288),   # q, k, v only
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"H{s['hidden']}-I{s['mlp']}-D{s['head_dim']}")
@pytest.mark.parametrize("T", [1, 2, 15, 16, 17, 32, 33])
def test_layer(shape, T):
    m = small_model(vocab=512, **shape)
    reqs = [W.RequestSpec(1, 3 + 9 * i) for i in range(T if T < 4 else T - 6)] + ([] if T < 4 else [W.RequestSpec(6, 21)])
    w = W.build_workload("few", m, reqs, n_kv_pages=T * 12 + 8, seed=1100 + T + m.hidden, std=0.02, resid_std=0.005)
    compare_layer(w, what=f"T={T} H{m.hidden} I{m.mlp_dim}")


@pytest.mark.parametrize("hidden", [512, 1024, 1536, 2560, 3072, 3584, 5120, 6144, 7168])
@pytest.mark.parametrize("T", [3, 16, 20])
def test_row_lengths(hidden, T):
    """Each length has a kernel of its own (2048, 4096 and 8192: above): ring depths of 2 to 14 requests, and 7, 8 and 10 above 4096."""
    m = small_model(64, 4, 2, hidden=hidden, mlp=288, vocab=512)
    w = W.build_workload("few", m, [W.RequestSpec(1, 3 + 9 * i) for i in range(T)], n_kv_pages=T * 14 + 8, seed=1500 + T + hidden, std=0.02,
                         resid_std=0.005)
    compare_layer(w, what=f"T={T} H{hidden}")


@pytest.mark.parametrize("hidden", [2048, 4096])
@pytest.mark.parametrize("T", [1, 16, 17, 32])
def test_layers_in_a_row(hidden, T):
    """(17 and 32 rows: q, k, v of the first layer alone, the layers behind it sum the split products' parts)"""
    m = small_model(64, 16, 4, hidden=hidden, mlp=1024, vocab=512)
    m.n_layers, m.page_size = 3, 16 if T % 2 else 32
    dw = W.build_deep_workload("few", m, [W.RequestSpec(1, 5 + 7 * i) for i in range(T)], n_kv_pages=T * 16 + 8, seed=1200 + T, std=0.02, resid_std=0.003)
    compare_deep(dw, f"few T={T}")


@pytest.mark.parametrize("hidden,mlp", [(2048, 12320), (3104, 8224), (1056, 608), (5120, 12320)])
@pytest.mark.parametrize("T", [3, 16])
def test_split_and_whole_products_in_a_row(hidden, mlp, T):
    """Down and output products that go whole or split by their rows, columns and contraction, layer behind layer."""
    m = small_model(64, 16, 4, hidden=hidden, mlp=mlp, vocab=512)
    m.n_layers = 2
    dw = W.build_deep_workload("few", m, [W.RequestSpec(1, 5 + 7 * i) for i in range(T)], n_kv_pages=T * 8 + 8, seed=1250 + T, std=0.02, resid_std=0.003)
    compare_deep(dw, f"few T={T} H{hidden} I{mlp}")


@pytest.mark.parametrize("projections", [("wdown",), ("wo",), ("wq", "wk", "wv"), ("wgate", "wup"), ("wv", "wdown"), ("wo", "wup")])
@pytest.mark.parametrize("T", [3, 16, 20])
def test_layers_with_adapters(projections, T):
    """Products that take their norm in beside products that an adapter's update goes into or behind.  (Left out, an update moves the
    output by 1e-2 to 1e-1 on average, five times the limit and more.)"""
    m = small_model(64, 16, 4, hidden=2048, mlp=1024, vocab=512)
    m.n_layers = 2
    dw = W.build_deep_workload("few_ad", m, [W.RequestSpec(1, 5 + 7 * i) for i in range(T)], n_kv_pages=T * 10 + 8, seed=1270 + T, std=0.02, resid_std=0.003)
    adapters = {0: W.make_adapter(m, 1270, 0, rank=16, projections=projections, scale=4.0, std=0.02),
                1: W.make_adapter(m, 1270, 1, rank=5, projections=projections[:1], scale=8.0, std=0.02)}
    compare_adapters(dw, adapters, [i % 3 - 1 for i in range(T)], f"few T={T}, adapters on {projections}")


def test_more_tiles_than_sums_are_kept_for():
    """33088 gate/up pairs: seventeen column tiles for most of 256 workgroups, which keep the sums of sixteen."""
    m = small_model(64, 4, 2, hidden=2048, mlp=33088, vocab=512)
    w = W.build_workload("few", m, [W.RequestSpec(1, 9), W.RequestSpec(2, 30)], n_kv_pages=8, seed=1300, std=0.02, resid_std=0.003)
    compare_layer(w, what="I33088")


@pytest.mark.parametrize("hidden,vocab", [(2048, 96), (2048, 4128), (2048, 131072), (4096, 8224), (4096, 16416), (512, 4128), (1536, 96), (3072, 4128),
                                          (3584, 4128)])
def test_logits(hidden, vocab):
    m = small_model(64, 4, 2, hidden=hidden, mlp=64, vocab=vocab)
    rng = np.random.default_rng(vocab)
    w = W.build_workload("few", m, [W.RequestSpec(1, 3)], n_kv_pages=4, seed=1400 + vocab, std=0.02, n_embeds=40)
    bits = O.bf16_encode(rng.standard_normal((40, hidden)).astype(np.float32))
    emb = O.EmbedPool(40, hidden)
    emb.write(np.arange(40, dtype=np.int32), bits)
    w_lm = O.bf16_decode(w.head.w_lm)
    ctx = make_ctx(w, max_dist_rows=33, max_top_k=16)
    ctx.embed_write(np.arange(40, dtype=np.int32), bits)
    for n in (1, 3, 16, 17, 32, 33):
        ids = rng.permutation(40)[:n].astype(np.int32)
        z = O.logits_from_embeds(m, w.head, emb, ids, True)
        gi, gp = ctx.get_next_dist(ids, 16, 1.0)
        zg = ctx.read_tap(TAP_LOGITS, n)
        # fp32 sums against 64 bits: 1e-5; besides, a normalised input that rounds the other way moves a row's logits by up to
        # one bf16 ulp of it (2^-7 of the largest, about 4.5) times a weight, and a row may hold two such inputs
        d = np.abs(zg - z)
        assert d.max() < 2 * 4.5 / 128 * np.abs(w_lm).max() and d.mean() < 1e-4, (n, d.max(), d.mean())
        oi, op = O.top_k_dist(zg.astype(np.float64), 16, 1.0)
        check_topk(gi, gp, zg.astype(np.float64), oi, op)
