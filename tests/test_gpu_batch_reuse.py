"""Batches deserialised one right after another, without a wait in between: each runs on its own copy of its arrays although
the host image they are built in is the same memory."""
import numpy as np
import pytest
import torch

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


def test_batches_whose_copies_wait_behind_queued_work_keep_their_own_arrays():
    """The stream has tens of milliseconds of work queued while the batches are created, so the first ones' copies are still
    to come when the host image is built anew: each runs on its own arrays."""
    w = W.c1_tiny()
    b = w.batch
    ctx = make_ctx(w)
    _, stored, want = gpu_forward(ctx, w)
    ctx.embed_write(b.in_embed_ids, w.embed_bits)  # (the in-place rows; waits for the stream, so before the queue fills)
    free = np.setdiff1d(np.arange(w.n_embeds, dtype=np.int32), b.in_embed_ids)
    a = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
    c = torch.mm(a, a)
    torch.cuda.synchronize()
    with torch.cuda.stream(ctx.stream):
        for _ in range(40):  # about a millisecond each
            torch.mm(a, a, out=c)
        queued = torch.cuda.Event()
        queued.record()
    outs, batches = [], []
    for k in range(3):
        out = b.out_embed_ids.copy()
        out[stored] = np.roll(free, k)[:len(stored)]
        outs.append(out)
        if k == 1:
            assert not queued.query()  # the first batch's copy has not begun
        batches.append(ctx.batch_create(clone_batch(b, out_embed_ids=out)))
    for out, pb in zip(outs, batches):
        ctx.forward(0, pb)
        assert np.array_equal(ctx.embed_read(out[stored]), want)


def test_a_captured_stream_is_refused_and_the_capture_goes_on():
    """batch_create during a capture is refused without ending it: the forward call recorded around it replays with the
    eager result, several times, with other work on the stream in between."""
    from paper_2510_24051_amd import PieError
    w = W.c1_tiny()
    b = w.batch
    ctx = make_ctx(w)
    stored = np.nonzero(b.out_embed_ids >= 0)[0]
    out = np.full_like(b.out_embed_ids, -1)
    out[stored] = np.setdiff1d(np.arange(w.n_embeds, dtype=np.int32), b.in_embed_ids)[:len(stored)]
    pb = ctx.batch_create(clone_batch(b, out_embed_ids=out))
    ctx.forward(0, pb)
    want = ctx.embed_read(out[stored])
    pb = ctx.batch_create(clone_batch(b, out_embed_ids=out))  # nothing has waited for this one's copy
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=ctx.stream):
        with pytest.raises(PieError) as e:
            ctx.batch_create(b)
        assert e.value.status == -6 and "captured" in str(e.value)
        ctx.forward(0, pb)
    for _ in range(3):
        ctx.embed_write(out[stored], np.zeros_like(want))
        with torch.cuda.stream(ctx.stream):
            graph.replay()
        assert np.array_equal(ctx.embed_read(out[stored]), want)
        ctx.batch_create(b).destroy()


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
