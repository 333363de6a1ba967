"""Batches deserialised one right after another, without a wait in between: each runs on its own copy of its arrays although
the host image they are built in is the same memory."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_forward, make_ctx
from helpers import clone_batch

pytestmark = pytest.mark.gpu


def test_batches_created_back_to_back_keep_their_own_arrays():
    w = W.c1_tiny()
    b = w.batch
    ctx = make_ctx(w)
    _, stored, want = gpu_forward(ctx, w)
    outs, batches = [], []
    free = np.setdiff1d(np.arange(w.n_embeds, dtype=np.int32), b.in_embed_ids)
    for k in range(3):  # the same requests, output rows elsewhere (the in-place requests too, so the inputs stay)
        out = b.out_embed_ids.copy()
        out[stored] = np.roll(free, k)[:len(stored)]
        outs.append(out)
        batches.append(ctx.batch_create(clone_batch(b, out_embed_ids=out)))
        if k == 0:
            ctx.embed_write(b.in_embed_ids, w.embed_bits)  # (the first forward call wrote the in-place rows)
    for out, pb in zip(outs, batches):
        ctx.forward(0, pb)
        got = ctx.embed_read(out[stored])
        assert np.array_equal(got, want)


def test_write_conflicts_are_found_across_calls():
    """The conflict check keeps its marks from call to call: a slot written by one batch is free for the next, and two
    tokens of one batch on one slot are refused every time."""
    from paper_2510_24051_amd import PieError
    w = W.c1_tiny()
    b = w.batch
    ctx = make_ctx(w)
    pages = np.array(b.page_ids).copy()
    n0 = int(b.page_indptr[1])
    pages[b.page_indptr[1]:b.page_indptr[1] + n0] = pages[:n0]
    kv = np.array(b.kv_len).copy()
    kv[1] = kv[0]
    clash = clone_batch(b, page_ids=pages, kv_len=kv)
    for _ in range(3):
        ctx.batch_create(b, validate=True).destroy()
        with pytest.raises(PieError) as e:
            ctx.batch_create(clash, validate=True)
        assert e.value.status == -4
