"""SwiGLU of exact sums is the same to the bit whichever kernel takes it: the epilogues of the products (a few rows, 32-row and
streamed and tiled ones) against the kernel that runs behind an adapter's update of gate and up, with an update of zero.

Every row of a gate or up weight has one value, so a sum is one product of two bf16 values in any order.  Rows are permutations of
multiples of 1/16 up to 3, whose squares add up exactly in 32 bits, so the norms in front agree as well.  Two forms of the
quotient that differ in the last of 24 bits show in about one of 10^5 activations, rounded to 8."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import make_ctx
from helpers import clone_batch
from paper_2510_24051_amd import TAP_ACT, Pie
from test_gpu_parity import small_model

pytestmark = pytest.mark.gpu


def one_value_a_row(rng, rows, cols):
    w = np.zeros((rows, cols), np.uint16)
    w[np.arange(rows), rng.integers(0, cols, rows)] = W.to_bf16_bits(2.0 * rng.standard_normal(rows))
    return w


@pytest.mark.parametrize("hidden,mlp,rows", [(2048, 8192, 5), (2048, 8192, 16), (2048, 8192, 60), (2048, 8192, 90), (2048, 8192, 300),
                                             (2048, 8192, 700), (512, 1024, 24), (512, 4096, 200), (1056, 4096, 150)])
def test_same_bits(hidden, mlp, rows):
    m = small_model(64, 4, 2, hidden=hidden, mlp=mlp)
    w = W.build_workload("swiglu", m, [W.RequestSpec(rows, 0)], n_kv_pages=rows // 16 + 4, seed=2100 + rows, with_head=False)
    rng = np.random.default_rng(rows)
    w.weights.wgate, w.weights.wup = one_value_a_row(rng, mlp, m.hidden), one_value_a_row(rng, mlp, m.hidden)
    w.weights.wo = np.zeros_like(w.weights.wo)
    values = W.to_bf16_bits(rng.integers(-48, 49, m.hidden) / 16.0)
    w.embed_bits = np.stack([rng.permutation(values) for _ in range(rows)])
    ctx = make_ctx(w)
    ctx.forward(0, ctx.batch_create(w.batch))
    ctx.synchronize()
    plain = ctx.read_tap(TAP_ACT, rows)
    b = clone_batch(w.batch, adapter_ids=np.zeros(1, np.int32))
    ctx2 = Pie(m, w.n_kv_pages, w.n_embeds, max_batch_tokens=rows, max_batch_requests=1, max_top_k=0, max_dist_rows=0, n_layers=1,
               max_adapters=1, max_lora_rank=16)
    ctx2.load_layer(0, w.weights)
    zero = (np.zeros((1, m.hidden), np.uint16), np.zeros((mlp, 1), np.uint16), 1.0)
    ctx2.load_adapter(0, [{"wgate": zero, "wup": zero}])
    ctx2.embed_write(b.in_embed_ids, w.embed_bits)
    ctx2.forward(0, ctx2.batch_create(b))
    ctx2.synchronize()
    updated = ctx2.read_tap(TAP_ACT, rows)
    print(f"    {rows} rows x {mlp}: {int((plain != updated).sum())} of {plain.size} activations differ", flush=True)
    assert len(np.unique(plain)) > 1000
    assert np.array_equal(plain, updated)
