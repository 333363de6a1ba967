"""Host paths around the batch's copy to the device, without a GPU: the library is loaded against a stand-in for the HIP
runtime (fake_hip.cpp: late copies, failures on request) in a process of its own, one per test."""
import os
import subprocess
import sys
from types import SimpleNamespace

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
MODEL = SimpleNamespace(hidden=128, n_q_heads=8, n_kv_heads=2, head_dim=64, mlp_dim=256, vocab=0, page_size=16, rms_eps=1e-5,
                        rope_theta=1e4)


def batch_of(reqs, first_page=0):
    """(new, prior) per request, pages in order from `first_page`."""
    tok = np.concatenate([[0], np.cumsum([n for n, _ in reqs])]).astype(np.int32)
    per = [(n + p + 15) // 16 for n, p in reqs]
    T = int(tok[-1])
    return SimpleNamespace(
        n_requests=len(reqs), n_tokens=T, tok_indptr=tok, in_embed_ids=np.arange(T), out_embed_ids=np.arange(T)[::-1],
        positions=np.concatenate([np.arange(p, p + n) for n, p in reqs]), page_indptr=np.concatenate([[0], np.cumsum(per)]),
        page_ids=first_page + np.arange(sum(per)), kv_len=np.array([n + p for n, p in reqs]), mask_indptr=None, mask_words=None,
        adapter_ids=None)


# ---- run in the child ------------------------------------------------------------------------
class Child:
    def __init__(self, fake):
        import ctypes as C
        import types
        self.C, self.fake = C, C.CDLL(fake, mode=C.RTLD_GLOBAL)
        for name, ret, args in (("fake_fail_new_at", None, [C.c_long]), ("fake_malloc_limit", None, [C.c_size_t]),
                                ("fake_largest_malloc", C.c_size_t, []), ("fake_copy_size", C.c_size_t, [C.c_int]),
                                ("fake_copy_data", C.c_void_p, [C.c_int]), ("fake_watch", None, [C.c_char_p, C.c_int]),
                                ("fake_launches", C.c_char_p, [])):
            getattr(self.fake, name).restype, getattr(self.fake, name).argtypes = ret, args
        sys.modules["torch"] = types.ModuleType("torch")  # (the binding keeps it for device tensors only)
        sys.path.insert(0, ROOT)
        from paper_2510_24051_amd import Pie, binding
        self.Pie, self.binding, self.lib = Pie, binding, binding.load_library()

    def context(self, n_pages=1024, tokens=256, requests=64, m=MODEL, adapters=0, rank=0, dist=(0, 0), layers=1):
        b, C = self.binding, self.C
        p = self.Pie.__new__(self.Pie)
        p.lib, p.device, p.stream, p.model, h = self.lib, None, None, m, C.c_void_p()
        md = b.ModelDescC(m.hidden, m.n_q_heads, m.n_kv_heads, m.head_dim, m.mlp_dim, m.vocab, m.page_size, m.rms_eps, m.rope_theta, layers)
        pd = b.PoolDescC(n_pages, 1024, tokens, requests, dist[1], dist[0], adapters, rank)
        assert self.lib.pie_create(C.byref(md), C.byref(pd), None, C.byref(h)) == 0
        p.ctx = h
        return p

    def loaded(self, pairs=(), m=MODEL, **kw):
        """A context with the weights of its layer and `pairs` (adapter, projection, rank)."""
        ctx, C = self.context(m=m, **kw), self.C
        room = np.zeros(2 * max(m.hidden, m.n_q_heads * m.head_dim) * max(m.mlp_dim, m.hidden, m.n_q_heads * m.head_dim), np.int8)
        at = C.c_void_p(room.ctypes.data)  # (kernels do nothing, copies read from here)
        for layer in range(kw.get("layers", 1)):
            assert self.lib.pie_load_layer(ctx.ctx, layer, *[at] * 9) == 0
        if m.vocab:
            head = np.zeros(m.vocab * m.hidden, np.int16)
            assert self.lib.pie_load_head(ctx.ctx, at, C.c_void_p(head.ctypes.data)) == 0
        for adapter, proj, r in pairs:
            for layer in range(kw.get("layers", 1)):
                assert self.lib.pie_load_adapter(ctx.ctx, adapter, layer, proj, r, C.c_float(1.0), at, at) == 0
        ctx.synchronize()  # (the copies are carried out here)
        return ctx

    def launches(self):
        return self.fake.fake_launches().decode().split("\n")[:-1]

    def copies(self):
        return [self.C.string_at(self.fake.fake_copy_data(i), self.fake.fake_copy_size(i)) for i in range(self.fake.fake_copies_done())]

    def status(self, fn):
        try:
            fn()
        except self.binding.PieError as e:
            return e.status, str(e)
        return 0, ""


def failed_wait(c):
    """A wait for the previous copy that fails leaves that copy in flight: the next call waits again before it writes."""
    ctx = c.context()
    a, b = batch_of([(1, 40), (20, 5)]), batch_of([(1, 90), (20, 33)], first_page=100)
    ctx.batch_create(a)
    ctx.synchronize()
    want = c.copies()[-1]
    n0 = len(c.copies())
    pa = ctx.batch_create(a)
    assert len(c.copies()) == n0  # still queued
    c.fake.fake_fail_event_syncs(1)
    assert c.status(lambda: ctx.batch_create(b))[0] == -6
    pb = ctx.batch_create(b)
    ctx.synchronize()
    assert c.copies()[n0] == want, "the image of a queued copy was rewritten"
    pa.destroy(), pb.destroy()


def late_copies(c):
    """Batches created one after another while every copy is still queued: each device block gets its own batch's image,
    also where the image has to grow in between."""
    ctx = c.context(n_pages=70000, tokens=64)
    batches = [batch_of([(1, 40 + k), (20, 5)], first_page=64 * k) for k in range(5)] + [batch_of([(1, 16 * 10000)] * 6), batch_of([(3, 7)])]
    want = []
    for b in batches:
        ctx.batch_create(b)
        ctx.synchronize()
        want.append(c.copies()[-1])
    assert len(want[5]) > len(want[4]) * 4
    c2 = c.context(n_pages=70000, tokens=64)  # (an image of its own, still small)
    n0 = len(c.copies())
    kept = [c2.batch_create(b) for b in batches]
    assert len(c.copies()) < n0 + len(batches)
    c2.synchronize()
    assert c.copies()[n0:] == want
    del kept


def captured_stream(c):
    """A call while the stream is captured is refused before the runtime is asked for anything else (a wait or an allocation
    would end the capture), and the context goes on as before."""
    ctx = c.context()
    a, big = batch_of([(1, 40)]), batch_of([(1, 16000)], first_page=8)
    pa = ctx.batch_create(a)  # its copy stays queued
    c.fake.fake_capturing(1)
    calls = c.fake.fake_event_syncs(), c.fake.fake_allocations()
    for b in (a, big):
        st, msg = c.status(lambda: ctx.batch_create(b))
        assert st == -6 and "captured" in msg, (st, msg)
    st, msg = c.status(lambda: ctx.batch_create(batch_of([(1, 16 * 2000)])))  # what is wrong with a batch is said first
    assert st == -2
    assert calls == (c.fake.fake_event_syncs(), c.fake.fake_allocations())
    c.fake.fake_capturing(0)
    ctx.batch_create(big).destroy()
    pa.destroy()


def failed_allocations(c):
    """Each C++ allocation of a first call in turn fails: the call reports it, and the next one makes the same batch."""
    b = batch_of([(1, 40), (2, 700), (20, 5), (1, 90)])
    first = c.context()
    pb = first.batch_create(b)
    want = pb.work(), pb.plan_info(), pb.prefill_work().tolist()
    failed = 0
    for k in range(1, 10000):
        ctx = c.context()
        c.fake.fake_fail_new_at(k)
        made = []
        st, _ = c.status(lambda: made.append(ctx.batch_create(b)))
        hit = c.fake.fake_new_failed()
        c.fake.fake_fail_new_at(0)
        for pb in made:
            pb.destroy()
        assert (st == -5) if hit else (st == 0), (k, st, hit)
        pb = ctx.batch_create(b)
        assert (pb.work(), pb.plan_info(), pb.prefill_work().tolist()) == want, k
        pb.destroy()
        ctx.close()
        if not hit:
            break
        failed += 1
    assert 20 < failed < 5000, failed


def failed_allocation_in_destroy(c):
    """pie_batch_destroy keeps device blocks for the next batch; it has no use for host memory to do so."""
    for n in (1, 12):  # fewer and more batches than blocks are kept
        ctx = c.context()
        pbs = [ctx.batch_create(batch_of([(1, 40)])) for _ in range(n)]
        for pb in pbs:
            c.fake.fake_fail_new_at(1)
            pb.destroy()
            c.fake.fake_fail_new_at(0)
        ctx.batch_create(batch_of([(1, 40)])).destroy()
        ctx.close()


def no_room_for_parts(c):
    """A device block that does not fit with the partial results is planned again without them: nothing cut, no wide groups,
    every page in a column group; without room for that either, PIE_ENOMEM, and the context goes on."""
    prompts, tree = batch_of([(33, 6000), (20, 9000), (1, 300)]), batch_of([(1, 16 * 1000 + 20)] * 96)
    own = 1000 + np.arange(96 * 2).reshape(96, 2)  # 96 requests on one prefix of 1000 pages, two pages of their own each
    tree.page_ids = np.concatenate([np.concatenate([np.arange(1000), pages]) for pages in own])
    page_bytes = MODEL.n_kv_heads * 2 * 16 * MODEL.head_dim * 2
    none = {"cut_blocks": 0, "most_parts": 1, "wide_groups": 0, "most_wide_parts": 1}
    for b, wide, alone in ((prompts, None, None), (tree, 3 * 1000 + 192, 24 * 1000 + 192)):  # pages asked for
        ctx = c.context(n_pages=1200, requests=128)
        c.fake.fake_largest_malloc()
        full = ctx.batch_create(b)
        parts, need = full.plan_parts(), c.fake.fake_largest_malloc()
        assert parts["cut_blocks"] + parts["wide_groups"] > 0
        c.fake.fake_malloc_limit(need - 1)
        small = ctx.batch_create(b)
        assert small.plan_parts() == none and c.fake.fake_largest_malloc() == need  # (asked for first)
        if wide:
            assert full.work()["kv_bytes_requested"] == wide * page_bytes and small.work()["kv_bytes_requested"] == alone * page_bytes
        c.fake.fake_malloc_limit(4096)
        assert c.status(lambda: ctx.batch_create(b))[0] == -5
        c.fake.fake_malloc_limit(1 << 62)
        again = ctx.batch_create(b)
        assert again.plan_parts() == parts
        for pb in (full, small, again):
            pb.destroy()
        ctx.close()


def adapter_updates_of_split_products(c):
    """Where the qkv or output product is split along K, an adapter's update joins the partial sums and no epilogue kernel runs in
    between: at the shapes of the device test of the same, all of which are split."""
    m = SimpleNamespace(**{**vars(MODEL), "hidden": 1024, "n_q_heads": 16, "n_kv_heads": 4, "mlp_dim": 512})
    c.fake.fake_watch(b"lora_up_kernel", 3)  # the kind of the destination
    batches = {153: [(70, 19), (1, 90), (45, 0), (1, 33), (2, 64), (1, 17), (33, 5)], 40: [(1, 11 + 3 * i) for i in range(40)],
               3: [(1, 20), (1, 1), (1, 300)]}
    for rows, projections in ((153, (0, 1, 2, 3)), (153, (2,)), (153, (3,)), (40, (0, 1, 3)), (3, (1, 3))):
        ctx = c.loaded([(0, pj, 20) for pj in projections], m, tokens=rows, requests=40, adapters=1, rank=32)
        b = batch_of(batches[rows])
        assert b.n_tokens == rows
        b.adapter_ids = np.zeros(b.n_requests, np.int32)
        pb = ctx.batch_create(b)
        c.launches()
        ctx.forward(0, pb)
        names = c.launches()
        kinds = [int(n.split()[1]) for n in names if "lora_up_kernel" in n]
        assert kinds == ([4] if min(projections) < 3 else []) + ([1] if 3 in projections else []), (rows, kinds)
        # neither product has an epilogue kernel (modes 0 and 1), and the second norm forms its rows from the partial sums
        assert not any("splitk_epilogue_kernelILi0E" in n or "splitk_epilogue_kernelILi1E" in n for n in names), names
        norms = [n for n in names if "rmsnorm_kernel" in n]
        assert len(norms) == 2 and "rmsnorm_kernelILi2E" in norms[1], norms
        pb.destroy()
        ctx.close()


def few_rows_with_an_adapter_on_o(c):
    """A few tokens at a width where the norms go into the products: with an adapter on the output projection that product leaves
    partial sums, so the second norm has to run; without one the products do everything."""
    m = SimpleNamespace(**{**vars(MODEL), "hidden": 2048, "n_q_heads": 32, "n_kv_heads": 8, "mlp_dim": 1024})
    for projections, norms in (((), 0), ((6,), 0), ((3,), 1), ((0, 3), 2)):
        ctx = c.loaded([(0, pj, 16) for pj in projections], m, tokens=16, adapters=1, rank=16)
        b = batch_of([(1, 20), (1, 1), (2, 300)])
        b.adapter_ids = np.zeros(b.n_requests, np.int32) if projections else None
        pb = ctx.batch_create(b)
        c.launches()
        ctx.forward(0, pb)
        names = c.launches()
        assert sum("rmsnorm_kernel" in n for n in names) == norms, (projections, names)
        assert any("rmsnorm_kernelILi2E" in n for n in names) == (3 in projections), (projections, names)
        pb.destroy()
        ctx.close()


def few_rows_by_width(c):
    """Which widths have their norms and rotary step inside the products, by the length of a row and the number of rows: every
    multiple of 512 up to 4096 at up to 16 rows, q, k, v of Embeds at up to 32, those of every multiple of 1024 up to 8192 at up to 16."""
    for hidden in (256, 480, 512, 768, 1024, 1536, 2048, 2560, 3072, 3584, 4096, 4608, 5120, 7168, 8192):
        m = SimpleNamespace(**{**vars(MODEL), "hidden": hidden, "n_q_heads": 4, "n_kv_heads": 2, "mlp_dim": 64})
        ctx = c.loaded(m=m, tokens=40)
        for tokens in (1, 16, 17, 32, 33):
            pb = ctx.batch_create(batch_of([(1, 20)] * tokens))
            c.launches()
            ctx.forward(0, pb)
            names = c.launches()
            fits = hidden % 512 == 0 and hidden <= 4096
            qkv = tokens <= 32 and fits or tokens <= 16 and hidden > 4096 and hidden % 1024 == 0
            assert any("few_rows_kernelILi0E" in n for n in names) == qkv != any("rope_append" in n for n in names), (hidden, tokens, names)
            assert any("few_rows_kernelILi2E" in n for n in names) == (fits and tokens <= 16), (hidden, tokens, names)
            assert sum("rmsnorm_kernel" in n for n in names) == 2 - qkv - (fits and tokens <= 16), (hidden, tokens, names)
            pb.destroy()
        ctx.close()


def few_rows_into_the_residual(c):
    """Output and down products of up to 16 rows: by themselves where the next kernel would not add split sums up for nothing (it takes
    its norm in, or there is none), else with most compute units at work and a contraction worth it; not for many long rows in few
    workgroups.  A table of (width, heads, mlp, tokens, adapter on, output product of each of two layers, down product of each)."""
    for hidden, heads, mlp, tokens, adapter, o, down in (
            (2048, 16, 1024, 16, None, 2, 2), (2048, 16, 1024, 17, None, 0, 0),       # norms inside: both, however short
            (1056, 16, 4096, 3, None, 0, 1), (3040, 64, 4096, 3, None, 0, 1),         # norms apart: only the last down product,
            (3104, 64, 8192, 3, None, 2, 2), (3104, 16, 1024, 3, None, 0, 1),         # long contractions in 194 workgroups,
            (4128, 32, 2048, 3, None, 2, 2), (4128, 16, 1024, 3, None, 0, 1),         # and in two column tiles a workgroup
            (3104, 64, 4096, 16, None, 2, 2), (3104, 64, 4128, 16, None, 2, 1), (3104, 64, 8224, 16, None, 2, 0), (1056, 16, 8224, 8, None, 0, 1),
            (2048, 16, 12288, 16, None, 2, 1), (2048, 16, 12320, 16, None, 2, 0), (2048, 16, 8224, 16, None, 2, 1), (2048, 16, 12320, 8, None, 2, 2),
            (3584, 16, 12320, 16, None, 2, 2), (5120, 64, 8192, 16, None, 2, 2), (5120, 64, 8224, 16, None, 2, 0), (6144, 64, 12320, 16, None, 2, 2),
            (2048, 16, 1024, 3, 3, 0, 2), (2048, 16, 1024, 3, 0, 2, 1), (2048, 16, 1024, 3, 4, 0, 2)):  # on o; q (its norm sums); gate
        m = SimpleNamespace(**{**vars(MODEL), "hidden": hidden, "n_q_heads": heads, "n_kv_heads": 8, "mlp_dim": mlp})
        ctx = c.loaded([] if adapter is None else [(0, adapter, 16)], m, tokens=32, adapters=1, rank=16, layers=2)
        b = batch_of([(1, 20)] * tokens)
        b.adapter_ids = None if adapter is None else np.zeros(tokens, np.int32)
        pb = ctx.batch_create(b)
        c.launches()
        ctx.forward_all(pb)
        names = c.launches()
        got = sum("few_stream_kernelILi1E" in n for n in names), sum("few_stream_kernelILi3E" in n for n in names)
        assert got == (o, down), (hidden, heads, mlp, tokens, adapter, got, names)
        pb.destroy()
        ctx.close()


def logits_of_few_rows(c):
    """Logits with their norm inside: up to 16 rows of every length that has a kernel, 17 to 32 rows of up to 3072, and of 4096 over
    many columns."""
    room = np.zeros(40 * 8, np.int32)
    out = c.C.c_void_p(room.ctypes.data)
    for hidden, vocab, most in ((512, 96, 32), (1000 // 32 * 32, 4096, 0), (3072, 512, 32), (3584, 32768, 16), (4096, 16384, 16), (4096, 16416, 32),
                                (5120, 512, 0)):
        m = SimpleNamespace(**{**vars(MODEL), "hidden": hidden, "mlp_dim": 64, "vocab": vocab})
        ctx = c.loaded(m=m, tokens=8, dist=(40, 8))
        for rows in (1, 16, 17, 32, 33):
            ids = np.arange(rows, dtype=np.int32)
            c.launches()
            assert c.lib.pie_get_next_dist(ctx.ctx, ids.ctypes.data_as(c.C.c_void_p), rows, 8, c.C.c_float(1.0), out, out) == 0
            names = c.launches()
            assert any("few_rows_kernelILi4E" in n for n in names) == (rows <= most) != any("rmsnorm" in n for n in names), (hidden, vocab, rows, names)
        ctx.close()


def stages_that_do_not_run(c):
    """A stage whose work a product has taken in reports 0, also when the call before it ran that stage."""
    m = SimpleNamespace(**{**vars(MODEL), "hidden": 2048, "n_q_heads": 32, "n_kv_heads": 8, "mlp_dim": 1024, "vocab": 512})
    ctx = c.loaded(m=m, tokens=40, dist=(40, 8))
    ctx.set_stage_timing(True)
    taken_in = {"norm1", "rope_append", "norm2"}
    for tokens, without in ((40, set()), (3, taken_in), (40, set()), (20, taken_in - {"norm2"})):
        pb = ctx.batch_create(batch_of([(1, 20 + i) for i in range(tokens)]))
        ctx.forward(0, pb)
        times = ctx.stage_times()
        ran = {"norm1", "qkv", "rope_append", "attn_decode", "attn_merge", "oproj", "norm2", "gateup", "down"} - without
        assert {k for k, v in times.items() if v > 0} - {"head_norm", "lm_head", "topk"} == ran, (tokens, times)
        pb.destroy()
    room = np.zeros(40 * 8, np.int32)
    out = c.C.c_void_p(room.ctypes.data)
    for rows, ran in ((40, True), (3, False)):
        ids = np.arange(rows, dtype=np.int32)
        assert c.lib.pie_get_next_dist(ctx.ctx, ids.ctypes.data_as(c.C.c_void_p), rows, 8, c.C.c_float(1.0), out, out) == 0
        times = ctx.stage_times()
        assert (times["head_norm"] > 0) == ran and times["lm_head"] > 0 and times["topk"] > 0, (rows, times)
    ctx.close()


def packed_prefill(c):
    """Batches without decode waves whose prompts have at most 64 (token, head) columns run them packed into as many waves as they fill,
    where that is fewer than a wave per head; not four heads or fewer of 128.  With a decode request in the batch the wave-per-head
    kernels run, once each, for the same blocks.  (The shapes of the device test of the same.)"""
    for D, G, new, prior, waves in ((128, 8, (3, 4), 1500, 1), (128, 8, (5, 8, 6, 7), 2500, 2), (128, 8, (8, 5), 2048, 2), (128, 8, (5, 8), 100, 2),
                                    (128, 8, (8, 9), 2500, 0), (64, 8, (5, 3, 4), 2048, 2), (64, 8, (4, 3), 90, 1), (64, 8, (8, 8), 3000, 2),
                                    (64, 4, (8, 8), 3000, 1), (64, 4, (13, 5, 16), 1777, 2), (64, 4, (16, 9, 5), 1300, 2), (64, 4, (16, 7), 100, 2),
                                    (64, 4, (8, 17), 2500, 0), (64, 2, (16,), 1200, 1), (64, 2, (9, 15), 110, 1), (64, 2, (9, 17), 2000, 0),
                                    (128, 4, (5, 8, 6, 7), 2500, 0), (128, 2, (9, 16, 12), 2000, 0)):
        m = SimpleNamespace(**{**vars(MODEL), "n_q_heads": 2 * G, "n_kv_heads": 2, "head_dim": D})
        ctx = c.loaded(m=m)
        prompts = [(n, prior // (1 + i)) for i, n in enumerate(new)]
        for decode in (False, True):
            pb = ctx.batch_create(batch_of(prompts + [(new[0], 0)] + ([(1, 700)] if decode else [])))
            assert (pb.plan_info()["decode_waves"] > 0) == decode
            c.launches()
            ctx.forward(0, pb)
            names = c.launches()
            packed = [n for n in names if "attn_packed" in n]
            plain = [n for n in names if "attn_prefill_kernel" in n and f"ELi{G}ELb0E" in n or "attn_both" in n]
            if waves and not decode:
                assert len(packed) == 1 and f"attn_packed_kernelILi{D}ELi{waves}E" in packed[0] and not plain, (D, G, new, names)
            else:
                assert not packed and len(plain) == 1, (D, G, new, decode, names)
            assert sum("attn_prefill_merge" in n for n in names) == (pb.plan_parts()["cut_blocks"] > 0), names
            assert any("attn_prefill_merge" in n for n in names) or prior <= 800, (D, G, new, prior)
            pb.destroy()
        ctx.close()


def attentions_in_one_launch(c):
    """Prompts of four query heads per kv head, or the tiles of a shared prefix, go with the decode waves in one launch; with stage
    timing on they are launched apart."""
    tree = batch_of([(1, 16 * 1000 + 20)] * 96)
    own = 1000 + np.arange(96 * 2).reshape(96, 2)
    tree.page_ids = np.concatenate([np.concatenate([np.arange(1000), pages]) for pages in own])
    for b, shared in ((batch_of([(150, 400), (1, 300), (1, 40)]), False), (tree, True)):
        ctx = c.loaded(n_pages=1200, requests=128)
        pb = ctx.batch_create(b)
        for timed in (False, True):
            ctx.set_stage_timing(timed)
            c.launches()
            ctx.forward(0, pb)
            names = [n for n in c.launches() if "attn_" in n and "merge" not in n]
            if timed:
                assert len(names) == 2 and not any("attn_both" in n for n in names), names
            else:
                assert len(names) == 1 and "attn_both_kernelILi64E" in names[0] and ("ELb1ELb1E" in names[0]) == shared, names
        pb.destroy()
        ctx.close()


CASES = {f.__name__: f for f in (failed_wait, late_copies, captured_stream, failed_allocations, failed_allocation_in_destroy, no_room_for_parts,
                                 adapter_updates_of_split_products, few_rows_with_an_adapter_on_o, few_rows_by_width, few_rows_into_the_residual,
                                 logits_of_few_rows, stages_that_do_not_run, packed_prefill, attentions_in_one_launch)}

if __name__ == "__main__":
    CASES[sys.argv[2]](Child(sys.argv[1]))
    print("case passed")
    sys.exit(0)


# ---- pytest ----------------------------------------------------------------------------------
@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-o", so, os.path.join(HERE, "fake_hip.cpp")], check=True)
    return so


@pytest.mark.parametrize("case", list(CASES))
def test_host_path(fake, case):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "case passed" in r.stdout, f"exit {r.returncode}\n{r.stdout}\n{r.stderr}"
