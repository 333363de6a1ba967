"""Decode requests that alias a long prefix, enough of them that the shared pages are walked in groups of up to 128 query
columns: the layer against the oracle, with bitmaps of every kind, private suffixes of different lengths, a second class
of two-token requests on the same prefix and a last group that is partly empty."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import compare_layer, hide_span, random_mask, small_model
from test_host_planner import requested_pages, sparse

pytestmark = pytest.mark.gpu


def sees_only_the_end(n_new, L, rng=None):
    m = W.causal_bitmap(n_new, L)
    m[:, :L - 20] = False
    return m


@pytest.mark.parametrize("head_dim,n_q,n_kv,R,pages", [(128, 32, 8, 150, 161), (64, 32, 16, 180, 250), (128, 64, 8, 60, 190)])
def test_long_shared_prefix_in_wide_groups(head_dim, n_q, n_kv, R, pages):
    m = small_model(head_dim, n_q, n_kv)
    rng = np.random.default_rng(R)
    P, prefix = 16, 16 * pages
    masks = [None, None, None, hide_span(3 * P + 5, 40 * P), random_mask(0.2), W.causal_bitmap, sees_only_the_end]
    reqs = [W.RequestSpec(1, prefix + int(rng.integers(0, 70)), prefix_group=0, prefix_len=prefix, mask=masks[i % 7], in_place=True)
            for i in range(R)]
    reqs += [W.RequestSpec(2, prefix + 9, prefix_group=0, prefix_len=prefix, mask=masks[i % 7]) for i in range(3)]
    reqs += [W.RequestSpec(1, 300), W.RequestSpec(20, 40)]
    w = W.build_workload("wide", m, reqs, n_kv_pages=pages + 6 * len(reqs) + 64, seed=900 + R, std=0.05)
    ctx, pb, _, _ = compare_layer(w, what=f"D{head_dim} G{n_q // n_kv} {R} branches on {prefix} tokens")
    assert pb.plan_parts()["wide_groups"] >= -(-R // (128 // (n_q // n_kv))) * n_kv
    work, page_bytes = pb.work(), n_kv * 2 * P * head_dim * 2
    G = n_q // n_kv
    private = sum(6 for _ in reqs) * page_bytes
    groups = -(-R // (128 // G)) + 3  # each shared page is asked for once per group of 128 columns
    assert work["kv_bytes_requested"] <= groups * pages * page_bytes + private + 2 * 20 * page_bytes


@pytest.mark.parametrize("head_dim,n_q,n_kv,R", [(128, 32, 8, 150), (64, 32, 16, 150)])
def test_wide_groups_over_masks_that_partly_overlap(head_dim, n_q, n_kv, R):
    """Every branch sees 60 pages of its own choice out of 400: most pages are walked by wide groups whose columns mostly do
    not see them, pages only one column group visits stay with it."""
    m = small_model(head_dim, n_q, n_kv)
    pages, seen = 400, sparse(np.random.default_rng(head_dim), R, 400, 60)

    def sees(own):
        def f(n_new, L, rng=None):
            mask = np.zeros((n_new, L), bool)
            for p in own:
                mask[:, p * 16:(p + 1) * 16] = True
            mask[:, pages * 16:] = True
            return mask
        return f
    reqs = [W.RequestSpec(1, pages * 16 + 39, prefix_group=0, prefix_len=pages * 16, mask=sees(own)) for own in seen]
    w = W.build_workload("overlap", m, reqs, n_kv_pages=pages + 3 * R + 8, seed=950 + head_dim, std=0.05)
    ctx, pb, _, _ = compare_layer(w, what=f"D{head_dim} G{n_q // n_kv} {R} branches, 60 of {pages} pages each")
    assert pb.plan_parts()["wide_groups"] == -(-R // (128 // (n_q // n_kv))) * n_kv
    families, cols, page_bytes = [(pages, 40, seen)], n_q // n_kv, n_kv * 2 * 16 * head_dim * 2
    assert requested_pages(families, cols, {0}) < requested_pages(families, cols, set())
    assert pb.work()["kv_bytes_requested"] == requested_pages(families, cols, {0}) * page_bytes
