"""Prefill attention of requests with few new tokens, whose (token, head) columns are packed into one or two waves: column counts
at and around a wave's 32 and at the limit of 64, both head sizes, every group size that packs, requests of different length in
one batch (the longest decides), whole blocks and blocks cut into parts, short contexts that go to the launch with weights as
pairs, pages of 32 tokens, and shapes on the other side of each limit.  A decode request beside them takes the batch back to a
wave per head: the same rows within rounding.  (Which shape is packed, and into how many waves: packed_prefill in
test_host_runtime_paths.py.)"""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_forward
from test_gpu_parity import compare_layer, random_mask, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,n_q,n_kv,new,prior,page", [
    (128, 16, 2, (3, 4), 1500, 16), (128, 16, 2, (5, 8, 6, 7), 2500, 16), (128, 16, 2, (8, 5), 2048, 32), (128, 16, 2, (5, 8), 100, 16),  # G = 8
    (128, 8, 1, (8, 9), 2500, 16),                                                            # 72 columns: not packed
    (64, 8, 1, (5, 3, 4), 2048, 16), (64, 8, 1, (4, 3), 90, 32), (64, 16, 2, (8, 8), 3000, 16),
    (64, 8, 2, (8, 8), 3000, 16), (64, 16, 4, (13, 5, 16), 1777, 16), (64, 8, 2, (16, 9, 5), 1300, 32), (64, 8, 2, (16, 7), 100, 16),  # G = 4
    (64, 8, 2, (8, 17), 2500, 16),                                                            # 68 columns: not packed
    (64, 4, 2, (16,), 1200, 16), (64, 4, 2, (9, 15), 110, 16), (64, 4, 2, (9, 17), 2000, 16),  # G = 2; 34 columns: not packed
    (128, 8, 2, (5, 8, 6, 7), 2500, 16), (128, 4, 2, (9, 16, 12), 2000, 16),                   # four and two heads of 128: not packed
])
def test_layer(head_dim, n_q, n_kv, new, prior, page):
    m = small_model(head_dim, n_q, n_kv)
    m.page_size = page
    reqs = [W.RequestSpec(n, prior // (1 + i)) for i, n in enumerate(new)]
    reqs += [W.RequestSpec(new[0], 0), W.RequestSpec(new[0], 40), W.RequestSpec(new[0], prior, mask=random_mask(0.3))]
    pages = sum((r.n_new + r.prior_len + page - 1) // page for r in reqs) + 8
    w = W.build_workload("packed", m, reqs, n_kv_pages=pages, seed=1500 + prior + new[0], std=0.05)
    ctx, pb, y_bits, _ = compare_layer(w, what=f"D{head_dim} G{n_q // n_kv} {new} new over {prior}")
    assert pb.plan_info()["prefill_workgroups"] > 0 and pb.plan_info()["decode_waves"] == 0
    assert (pb.plan_parts()["cut_blocks"] > 0) == (prior > 800)
    _, _, again = gpu_forward(ctx, w)  # the partial results are reused: the same bits
    assert np.array_equal(np.asarray(y_bits), np.asarray(again))


@pytest.mark.parametrize("head_dim,n_q,n_kv", [(64, 8, 2), (128, 16, 2), (128, 8, 2)])
def test_beside_a_decode_request(head_dim, n_q, n_kv):
    m = small_model(head_dim, n_q, n_kv)
    reqs = [W.RequestSpec(6, 2000), W.RequestSpec(1, 700), W.RequestSpec(8, 90)]
    w = W.build_workload("packed", m, reqs, n_kv_pages=190, seed=1600, std=0.05)
    _, pb, _, _ = compare_layer(w, what="6 and 8 new beside a decode request")
    assert pb.plan_info()["decode_waves"] > 0
