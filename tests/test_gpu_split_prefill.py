"""Prefill attention whose query blocks are cut into parts (few blocks over long contexts): the whole layer against the
oracle, for every group size the kernel is built for, with causal, bitmap and short requests in one batch, so that cut and
whole blocks, empty rows and parts of unequal length meet."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_forward
from test_gpu_parity import compare_layer, random_mask, small_model

pytestmark = pytest.mark.gpu


def nothing_before(first):
    """Only keys from index `first` on: whole parts of a block see nothing."""
    def f(n_new, L, rng=None):
        m = W.causal_bitmap(n_new, L)
        m[:, 16:first] &= False
        m[0, :] = False  # and one row without any key
        return m
    return f


@pytest.mark.parametrize("head_dim,n_q,n_kv,new,prior", [(128, 8, 2, 7, 1500), (64, 8, 2, 45, 1111), (128, 8, 1, 33, 1300),
                                                         (64, 4, 2, 64, 2047), (128, 2, 2, 32, 1024), (64, 8, 1, 3, 4000)])
def test_cut_query_blocks_match(head_dim, n_q, n_kv, new, prior):
    m = small_model(head_dim, n_q, n_kv)
    reqs = [W.RequestSpec(new, prior), W.RequestSpec(40, 0), W.RequestSpec(1, 90), W.RequestSpec(new, prior // 2),
            W.RequestSpec(new + 2, prior, mask=random_mask(0.3)), W.RequestSpec(40, prior, mask=nothing_before(prior - 30)),
            W.RequestSpec(33, prior, mask=random_mask(0.01))]
    pages = sum((r.n_new + r.prior_len + 15) // 16 for r in reqs) + 8
    w = W.build_workload("cut", m, reqs, n_kv_pages=pages, seed=700 + prior, std=0.05)
    ctx, pb, y_bits, _ = compare_layer(w, what=f"D{head_dim} G{n_q // n_kv} {new} new over {prior}")
    parts = pb.plan_parts()
    assert parts["cut_blocks"] > 0 and parts["most_parts"] > 1, parts
    _, _, again = gpu_forward(ctx, w)  # the partial results are reused: the same bits
    assert np.array_equal(np.asarray(y_bits), np.asarray(again))
