"""Batches whose prefill (or shared-prefix) workgroups and decode waves share one launch: fewer and more of either kind than
the 256 of a chunk, query blocks cut along their pages, both head dimensions; and the same batch with stage timing on, which
keeps the kernels apart.  (Shared groups: the batches of wide groups run this way.)"""
import numpy as np
import pytest

import workloads as W

from test_gpu_parity import compare_layer, small_model

pytestmark = pytest.mark.gpu


def requests(prompts, prompt, prior, decode, context):
    return [W.RequestSpec(prompt, prior + 9 * i) for i in range(prompts)] + [W.RequestSpec(1, context + 5 * i) for i in range(decode)]


@pytest.mark.parametrize("D,n_kv,shape,workgroups,waves", [
    (128, 2, (2, 140, 0, 5, 60), 16, 14),            # a handful of each
    (64, 8, (1, 1200, 3, 7, 40), 288, 64),           # more prefill workgroups than a chunk
    (64, 8, (2, 150, 90, 64, 300), 80, 1896),        # more decode workgroups (of four waves) than a chunk
    (128, 2, (6, 170, 400, 100, 200), 72, 1450),
    (128, 4, (3, 40, 2600, 12, 500), 24, 408),       # few query blocks over long contexts: cut into parts, 264 workgroups
    (64, 4, (3, 7, 2600, 12, 500), 16, 408),
])
def test_prefill_and_decode_in_one_launch(D, n_kv, shape, workgroups, waves):
    m = small_model(D, 4 * n_kv, n_kv, hidden=256, mlp=256, vocab=512)
    reqs = requests(*shape)
    pages = sum((r.n_new + r.prior_len + 15) // 16 for r in reqs) + 8
    w = W.build_workload("both", m, reqs, n_kv_pages=pages, seed=sum(shape) + D, std=0.02, resid_std=0.01)
    ctx, pb, y, _ = compare_layer(w, what=f"D={D} {shape}")
    info, parts = pb.plan_info(), pb.plan_parts()
    assert (info["prefill_workgroups"], info["decode_waves"]) == (workgroups, waves)
    assert (parts["most_parts"] > 1) == (shape[2] > 2000), parts
    ctx.set_stage_timing(True)  # the same kernels' work, launched apart: the same results bit for bit
    ctx.forward(0, pb)
    assert np.array_equal(ctx.embed_read(w.batch.out_embed_ids), y)


@pytest.mark.parametrize("D,n_q,n_kv,R,pages,prompt", [
    (128, 32, 8, 150, 161, False),   # tiles of groups of 32 requests beside the decode waves of their own pages
    (64, 32, 16, 150, 250, True),    # two query heads per kv head; a prompt whose rows see few keys keeps a launch of its own
])
def test_shared_prefix_and_decode_in_one_launch(D, n_q, n_kv, R, pages, prompt):
    m = small_model(D, n_q, n_kv)
    rng = np.random.default_rng(R + D)
    prefix = 16 * pages
    reqs = [W.RequestSpec(1, prefix + int(rng.integers(1, 90)), prefix_group=0, prefix_len=prefix) for _ in range(R)]
    reqs += [W.RequestSpec(1, 300)] + ([W.RequestSpec(20, 3)] if prompt else [])
    w = W.build_workload("both_shared", m, reqs, n_kv_pages=pages + 8 * len(reqs) + 64, seed=700 + D, std=0.05)
    ctx, pb, y, _ = compare_layer(w, what=f"D={D} {R} branches on {prefix} tokens")
    info, parts = pb.plan_info(), pb.plan_parts()
    # wide groups and decode waves, and no prompt of plain weights that would take the joint launch instead
    assert parts["wide_groups"] > 0 and info["decode_waves"] > 0 and info["prefill_workgroups"] == 0, (info, parts)
    assert (info["prefill_workgroups_pair_weights"] > 0) == prompt
    ctx.set_stage_timing(True)  # launched apart
    ctx.forward(0, pb)
    assert np.array_equal(ctx.embed_read(w.batch.out_embed_ids), y)
