"""get_next_dist over logits of every shape: hidden states that pick one column of the LM head each make the logits of a row
exactly that column's bf16 values, so ids have to be exact (equal logits in the order of their ids) and probabilities those of
a float64 softmax; for every size of the groups whose maxima the selection starts from, ragged last chunks, and the sizes that
are left to the chunk kernels."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import make_ctx
from oracle import pie_oracle as O
from test_gpu_parity import small_model

pytestmark = pytest.mark.gpu


def columns(V, rng):
    normal = rng.standard_normal(V).astype(np.float32)
    one_group = normal - 20
    one_group[5000 % V:5000 % V + 700] = 3 + rng.random(700).astype(np.float32)[:len(one_group[5000 % V:5000 % V + 700])]  # the top within one chunk
    few = np.round(normal * 2) / 2                          # a handful of values, thousands of ties each
    outlier = normal.copy()
    outlier[rng.integers(0, V, 3)] = [1e30, 3e5, -1e30]     # a range of keys that a first histogram does not resolve
    both = np.where(rng.random(V) < 0.5, -1e-30, 1e-30).astype(np.float32) * rng.integers(1, 200, V)
    masked = np.where(rng.random(V) < 0.9, -np.inf, normal).astype(np.float32)
    return {"normal": normal, "constant": np.full(V, 0.5, np.float32), "ascending": np.linspace(-4, 4, V, dtype=np.float32),
            "descending": np.linspace(4, -4, V, dtype=np.float32), "one group": one_group, "few values": few, "outliers": outlier,
            "tiny": both, "negative": -np.abs(normal) - 1, "zeros of both signs": np.where(rng.random(V) < 0.5, -0.0, 0.0).astype(np.float32),
            "masked": masked}


@pytest.mark.parametrize("V,ks", [(131072, (1, 2, 3, 5, 8, 17, 33, 64, 100, 256, 300, 512, 700, 1024)), (128256, (4, 50, 256)),
                                  (32000, (1, 7, 50, 256, 512, 1000)), (8224, (1, 16, 100, 257)), (8192, (2, 256)), (1024, (1, 8, 32, 512, 1024)),
                                  (96, (1, 3, 96))])
def test_ids_are_exact_and_probabilities_those_of_a_softmax(V, ks):
    rng = np.random.default_rng(V)
    m = small_model(hidden=128, vocab=V)
    w = W.build_workload("topk", m, [W.RequestSpec(1, 3)], n_kv_pages=4, seed=9, std=0.05, n_embeds=32)
    cols = columns(V, rng)
    n = len(cols)
    with np.errstate(over="ignore"):
        bits = np.stack([O.bf16_encode(np.where(np.isneginf(c), 0, c).astype(np.float32)) for c in cols.values()], axis=1)
    neg = np.stack([np.isneginf(c) for c in cols.values()], axis=1)
    logits = O.bf16_decode(bits).astype(np.float32)
    w.head.g_final = None
    w.head.w_lm = np.zeros((V, m.hidden), np.uint16)
    w.head.w_lm[:, :n] = bits
    # a logit of -inf cannot be made by finite weights (0 x inf): the largest finite negative stands for it, far below the rest
    w.head.w_lm[:, :n][neg] = O.bf16_encode(np.full(1, -2e38, np.float32))[0]
    logits[neg] = O.bf16_decode(O.bf16_encode(np.full(1, -2e38, np.float32)))[0]
    ctx = make_ctx(w, max_dist_rows=n, max_top_k=max(ks))
    ids = np.arange(n, dtype=np.int32)
    ctx.embed_write(ids, O.bf16_encode(np.eye(n, m.hidden, dtype=np.float32)))
    z = logits.T.astype(np.float64)
    order = np.argsort(-z, axis=1, kind="stable")
    for k in ks:
        for temperature in (1.0, 0.7):
            gi, gp = ctx.get_next_dist(ids, k, temperature)
            with np.errstate(under="ignore"):
                zz = (z - z.max(1, keepdims=True)) / temperature
                p = np.exp(zz) / np.exp(zz).sum(1, keepdims=True)
            for r, name in enumerate(cols):
                what = f"V={V} k={k} T={temperature} {name}"
                want = order[r, :k]
                if name == "zeros of both signs":  # +0 and -0 are equal numbers, their order is free
                    assert len(set(gi[r])) == k, what
                else:
                    assert np.array_equal(gi[r], want), what
                # fp32: the sum of up to 131072 terms in groups (1e-6), the base-2 exponential of a scaled argument up to 8 (2e-6)
                np.testing.assert_allclose(gp[r], p[r, gi[r]], rtol=1e-5, atol=1e-37, err_msg=what)
