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


def logit_context(cols, V, ks, rows):
    """A context whose Embed j makes the logits of cols[j] (bf16 values), and 2 x as an Embed twice those."""
    m = small_model(hidden=128, vocab=V)
    w = W.build_workload("topk", m, [W.RequestSpec(1, 3)], n_kv_pages=4, seed=9, std=0.05, n_embeds=rows)
    w.head.g_final = None
    w.head.w_lm = np.zeros((V, m.hidden), np.uint16)
    w.head.w_lm[:, :len(cols)] = np.stack([O.bf16_encode(np.asarray(c, np.float32)) for c in cols], axis=1)
    return m, make_ctx(w, max_dist_rows=rows, max_top_k=max(ks))


def tied_columns(V, rng):
    """Rows whose selection cannot stop at a few more than k logits, or whose values crowd in a part of their range."""
    normal = rng.standard_normal(V).astype(np.float32)
    top = np.minimum(normal, 3.0)
    top[rng.permutation(V)[:V // 4]] = 4.0                      # a quarter ties for the first places but a few
    top[rng.integers(0, V, 5)] = 4.5
    above = -np.abs(normal) - 1
    above[rng.integers(0, V)] = 20                              # one far above all others
    group = normal - 20
    group[V // 3:V // 3 + 700] = 3 + rng.random(len(group[V // 3:V // 3 + 700]))
    return {"normal": normal, "constant": np.full(V, 0.5), "unwritten": np.zeros(V), "two values": np.where(normal > 0, 1.0, -1.0),
            "quarter tied": top, "half steps": np.round(normal * 2) / 2, "one above": above, "one group": group,
            "tied at the end": np.where(np.arange(V) >= V - V // 8, 2.0, 1.0), "blocks": np.repeat(rng.standard_normal((V + 63) // 64), 64)[:V],
            "few left": np.where(rng.random(V) < 0.9995, -2e38, normal), "eighths": np.round(normal * 8) / 8}


@pytest.mark.parametrize("V,ks", [(131072, (1, 2, 5, 50, 256, 511, 1024)), (128256, (3, 50, 256, 1000)), (32000, (1, 20, 256, 1000)), (8192, (1, 31, 256)),
                                  (12320, (1, 100, 385))])
def test_equal_and_crowded_logits(V, ks):
    rng = np.random.default_rng(V + 1)
    cols = tied_columns(V, rng)
    m, ctx = logit_context(list(cols.values()), V, ks, len(cols))
    ids = np.arange(len(cols), dtype=np.int32)
    ctx.embed_write(ids, O.bf16_encode(np.eye(len(cols), m.hidden, dtype=np.float32)))
    z = np.stack([O.bf16_decode(O.bf16_encode(np.asarray(c, np.float32))) for c in cols.values()]).astype(np.float64)
    order = np.argsort(-z, axis=1, kind="stable")
    with np.errstate(under="ignore"):
        p = np.exp(z - z.max(1, keepdims=True))
        p /= p.sum(1, keepdims=True)
    for k in ks:
        gi, gp = ctx.get_next_dist(ids, k, 1.0)
        for r, name in enumerate(cols):
            assert np.array_equal(gi[r], order[r, :k]), f"V={V} k={k} {name}"
            np.testing.assert_allclose(gp[r], p[r, gi[r]], rtol=1e-5, atol=1e-37, err_msg=f"V={V} k={k} {name}")


@pytest.mark.parametrize("V,k", [(128256, 50), (128256, 256), (32000, 256)])
def test_a_row_of_equal_logits_takes_little_longer(V, k):
    """An Embed that nobody wrote is zero and makes all logits equal; one such row must not set the time of the call.  Top-k
    over 16 rows with one such row, or one whose values crowd in another way, against 16 ordinary rows, medians of 20 passes:
    2 to 3 times as long at most (the chunk kernels too).  A selection that takes every group that reaches the bound, and counts equal
    logits one by one in every refinement, takes 8 to 40 times as long."""
    cols = tied_columns(V, np.random.default_rng(V))
    m, ctx = logit_context(list(cols.values()), V, [k], 16)
    ids = np.arange(16, dtype=np.int32)
    ctx.set_stage_timing(True)

    def median_ms(name):
        x = np.zeros((16, m.hidden), np.float32)
        x[:, list(cols).index("normal")] = 1
        if name != "normal":
            x[3], x[3, list(cols).index(name)] = 0, 1
        ctx.embed_write(ids, O.bf16_encode(x))
        times = []
        for _ in range(20):
            ctx.get_next_dist(ids, k, 1.0)
            times.append(ctx.stage_times()["topk"])
        return float(np.median(times))

    median_ms("normal")
    plain = median_ms("normal")
    for name in ("constant", "unwritten", "two values", "quarter tied", "half steps", "few left", "one above", "one group"):
        t = median_ms(name)
        print(f"  V={V} k={k} {name}: {t * 1e3:.1f} us, ordinary rows {plain * 1e3:.1f}", flush=True)
        assert t <= 4 * plain, name


def test_infinite_and_undefined_logits():
    """-inf among the logits (a mask) is below everything and adds nothing; a row of -inf alone, of +inf or of NaN has no distribution,
    but the call returns, with ids of the vocabulary or -1."""
    V, k = 32000, 64
    rng = np.random.default_rng(3)
    normal = rng.standard_normal(V).astype(np.float32)
    low = -2e38  # twice that is -inf in fp32
    cols = [np.where(rng.random(V) < 0.9, low, normal), np.where(np.arange(V) < V - 80, low, normal), np.full(V, low), np.where(rng.random(V) < 0.01, 2e38, normal)]
    m, ctx = logit_context(cols, V, [k], 6)
    x = np.zeros((6, m.hidden), np.float32)
    for j in range(len(cols)):
        x[j, j] = 2
    bits = O.bf16_encode(x)
    bits[4, 0] = 0x7FC0                   # every logit NaN
    ids = np.arange(6, dtype=np.int32)
    ctx.embed_write(ids, bits)
    gi, gp = ctx.get_next_dist(ids, k, 1.0)  # (row 5 is an Embed of zeros)
    for r in (0, 1):
        z = 2 * O.bf16_decode(O.bf16_encode(cols[r])).astype(np.float64)
        z[z < -3.4e38] = -np.inf
        order = np.argsort(-z, kind="stable")[:k]
        p = np.exp(z - z.max())
        assert np.array_equal(gi[r], order)
        np.testing.assert_allclose(gp[r], (p / p.sum())[order], rtol=1e-5)
    assert np.array_equal(gi[2], np.arange(k)) and np.array_equal(np.sort(gi[3]), np.nonzero(cols[3] > 1e38)[0][:k])
    assert np.array_equal(gi[5], np.arange(k)) and np.allclose(gp[5], 1 / V, rtol=1e-5)
    assert ((gi >= -1) & (gi < V)).all() and np.isnan(gp[4]).all()
    for n in (1, 4):  # and an ordinary row beside them is untouched
        ctx.embed_write(ids[:1], O.bf16_encode(np.eye(1, m.hidden, 3, dtype=np.float32)))
        gi1, _ = ctx.get_next_dist(ids[:n], k, 1.0)
        z = O.bf16_decode(O.bf16_encode(cols[3])).astype(np.float64)
        assert np.array_equal(gi1[0], np.argsort(-z, kind="stable")[:k])


def test_the_sum_over_far_groups_keeps_the_precision_of_expf():
    """One logit 7 to 10 above 128255 equal ones, so that the sum is made of other groups' shares: the top probability against
    64 bits, on average.  expf is off by up to one ulp (1.2e-7), by a quarter of that on average; the sums, the reciprocal and the
    smallest terms added to 1 one by one (15 times 6e-8, of a sum of at least 6.8) add 3e-8 to 5e-8; a base-2 exponential of
    the scaled distance is off by 2e-7 on average here (its argument, around 13, is rounded to a multiple of 2^-20)."""
    V, gaps = 128256, np.arange(7 * 16, 10 * 16) / 16.0
    at = np.random.default_rng(3).integers(0, V, len(gaps))
    cols = np.zeros((len(gaps), V), np.float32)
    cols[np.arange(len(gaps)), at] = gaps
    m, ctx = logit_context(cols, V, (50,), len(gaps))
    ids = np.arange(len(gaps), dtype=np.int32)
    ctx.embed_write(ids, O.bf16_encode(np.eye(len(gaps), m.hidden, dtype=np.float32)))
    gi, gp = ctx.get_next_dist(ids, 50, 1.0)
    assert np.array_equal(gi[:, 0], at)
    off = np.abs(gp[:, 0].astype(np.float64) * (1 + (V - 1) * np.exp(-gaps)) - 1)
    assert off.mean() < 1.2e-7, (off.max(), off.mean())
