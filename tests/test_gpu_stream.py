"""Products at 1 to 640 rows on the streaming kernel: every form it has (rows of a tile, K slices inside a workgroup),
whole and split along K, one to eight row tiles, at row counts around the tiles' edges, with output widths that leave the last
column tile partly empty and contractions of an odd number of 64-wide steps; through LM heads (every logit) and through
layers (all four epilogues, partial sums left to the following kernels)."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import make_ctx
from helpers import check_topk
from oracle import pie_oracle as O
from paper_2510_24051_amd import TAP_LOGITS, product_stream
from test_gpu_model import compare_deep
from test_gpu_parity import compare_layer, small_model

pytestmark = pytest.mark.gpu


def workspace(m, rows):  # partial sums a context of that many batch tokens has room for
    qkv = (m.n_q_heads + 2 * m.n_kv_heads) * m.head_dim
    return min(rows, 256) * max(2 * m.mlp_dim, (max(qkv, m.hidden) + 31) // 32 * 32) * 8


def form(m, rows, n_out, k):
    return tuple(product_stream(rows, n_out, k, workspace(m, rows)).values())


@pytest.mark.parametrize("hidden,vocab,mlp,rows", [
    (2048, 12320, 320, {1: (64, 4, 1), 33: (64, 4, 1), 64: (64, 4, 1), 65: (96, 4, 1), 96: (96, 4, 1)}),
    (1024, 24608, 320, {5: (64, 2, 1), 64: (64, 2, 1), 96: (96, 2, 1), 97: (128, 2, 1), 257: (160, 1, 1), 320: (160, 1, 1), 384: (192, 1, 1)}),
    (2048, 32992, 320, {1: (64, 1, 1), 64: (64, 1, 1)}),
    (4096, 16416, 4096, {33: (64, 1, 3), 97: (128, 1, 3), 129: (160, 1, 3), 192: (192, 1, 3)}),
    (2048, 8224, 320, {192: (64, 2, 1), 256: (96, 2, 1), 320: (128, 2, 1)}),
    (1088, 32992, 320, {129: (160, 1, 1), 161: (192, 1, 1)}),  # seventeen k steps
    (2048, 40992, 320, {97: (128, 1, 1), 128: (128, 1, 1)}),
    (4096, 8224, 4096, {65: (96, 2, 3), 128: (128, 2, 3)}),
    (4096, 12320, 4096, {129: (160, 2, 2)}),
])
def test_lm_heads(hidden, vocab, mlp, rows):
    m = small_model(64, 4, 2, hidden=hidden, mlp=mlp, vocab=vocab)
    most = max(rows)
    w = W.build_workload("stream", m, [W.RequestSpec(1, 3)], n_kv_pages=4, seed=800 + hidden + vocab, std=0.02, n_embeds=most)
    emb = O.EmbedPool(most, m.hidden)
    rng = np.random.default_rng(vocab)
    all_ids = rng.permutation(most).astype(np.int32)
    bits = O.bf16_encode(rng.standard_normal((most, m.hidden)).astype(np.float32))
    emb.write(all_ids, bits)
    w_lm = O.bf16_decode(w.head.w_lm)
    z = O.logits_from_embeds(m, w.head, emb, all_ids, True)
    for n, want in rows.items():
        ctx = make_ctx(w, max_dist_rows=n, max_top_k=16)  # (the workspace grows with the rows a context takes)
        ctx.embed_write(all_ids, bits)
        assert form(m, n, vocab, hidden) == want, n
        gi, gp = ctx.get_next_dist(all_ids[:n], 16, 1.0)
        zg = ctx.read_tap(TAP_LOGITS, n)
        # fp32 sums against 64 bits: 1e-5; besides, a normalised input that rounds the other way moves a row's logits by up to
        # one bf16 ulp of it (2^-7 of the largest, about 4.5) times a weight, and a row may hold two such inputs
        d = np.abs(zg - z[:n])
        assert d.max() < 2 * 4.5 / 128 * np.abs(w_lm).max() and d.mean() < 1e-4, (n, d.max(), d.mean())
        oi, op = O.top_k_dist(zg.astype(np.float64), 16, 1.0)
        check_topk(gi, gp, zg.astype(np.float64), oi, op)
        del ctx


def mixed(T, n_decode):
    if T <= n_decode:
        return [W.RequestSpec(1, 3 + 5 * i) for i in range(T)]
    return [W.RequestSpec(1, 3 + 5 * i) for i in range(n_decode)] + [W.RequestSpec(T - n_decode, 19)]


@pytest.mark.parametrize("T,shape,forms", [
    (1, dict(hidden=2048, mlp=8192), {"gateup": (64, 4, 1)}),
    (64, dict(hidden=2048, mlp=8192), {"gateup": (64, 4, 1)}),
    (96, dict(hidden=2048, mlp=8192), {"gateup": (96, 4, 1), "down": (96, 4, 8)}),
    (192, dict(hidden=2048, mlp=8192), {"gateup": (96, 2, 1), "down": (96, 2, 8)}),
    (300, dict(hidden=2048, mlp=8192), {"gateup": (160, 2, 1)}),
    (65, dict(hidden=2048, mlp=8224), {"gateup": (96, 2, 1)}),
    (128, dict(hidden=2048, mlp=8224), {"gateup": (128, 2, 1)}),
    (157, dict(hidden=2048, mlp=8224), {"gateup": (160, 2, 1)}),
    (129, dict(hidden=1024, mlp=16448), {"gateup": (160, 1, 1)}),
    (192, dict(hidden=1024, mlp=16448), {"gateup": (192, 1, 1)}),
    (96, dict(head_dim=128, n_q=32, n_kv=8, hidden=4096, mlp=4096),
     {"qkv": (96, 2, 4), "o": (96, 4, 4), "gateup": (96, 2, 4), "down": (96, 4, 4)}),
    (200, dict(head_dim=128, n_q=64, n_kv=8, hidden=2048, mlp=512), {"qkv": (96, 2, 1)}),
    # several row tiles of small products
    (300, dict(hidden=2048, mlp=8192), {"qkv": (64, 4, 1), "o": (64, 4, 1)}),
    (260, dict(hidden=1024, mlp=4096), {"qkv": (64, 4, 1), "gateup": (96, 2, 1)}),
    (420, dict(hidden=1024, mlp=4096), {"o": (64, 4, 1), "gateup": (64, 1, 1)}),
    (500, dict(hidden=1024, mlp=4096), {"gateup": (128, 2, 1)}),
    (500, dict(n_q=32, n_kv=8, hidden=2048, mlp=512), {"qkv": (64, 2, 1), "o": (64, 4, 1), "gateup": (64, 4, 1), "down": (64, 2, 1)}),
    (640, dict(hidden=1024, mlp=512), {"qkv": (96, 4, 1), "down": (96, 2, 1)}),
    (129, dict(hidden=1024, mlp=16448), {"down": (64, 1, 15)}),
])
def test_layers(T, shape, forms):
    m = small_model(**{**dict(head_dim=64, n_q=16, n_kv=4), **shape}, vocab=512)
    H, D = m.hidden, m.head_dim
    sizes = {"qkv": ((m.n_q_heads + 2 * m.n_kv_heads) * D, H), "o": (H, m.n_q_heads * D), "gateup": (2 * m.mlp_dim, H), "down": (H, m.mlp_dim)}
    assert {k: form(m, T, *sizes[k]) for k in forms} == forms
    w = W.build_workload("stream", m, mixed(T, 20), n_kv_pages=T // 16 + 240, seed=900 + T, std=0.02, resid_std=0.005)
    compare_layer(w, what=f"T={T} H{H} I{m.mlp_dim}")


def test_down_projection_partials_carried_to_the_next_layer():
    m = small_model(64, 16, 4, hidden=2048, mlp=8192, vocab=512)
    m.n_layers = 2
    assert form(m, 192, m.hidden, m.mlp_dim) == (96, 2, 8)
    dw = W.build_deep_workload("carried", m, mixed(192, 20), n_kv_pages=252, seed=930, std=0.02, resid_std=0.003)
    compare_deep(dw, "carried T=192")
