"""Layer products at up to 32 rows with each column block's contraction cut in two slices inside the workgroup: even and odd
numbers of 128-wide iterations (the odd ones stay whole), splits whose last part is shorter, ragged rows."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import compare_layer, small_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,mlp", [(256, 1280), (384, 2816), (1152, 1024), (1024, 3328)])
@pytest.mark.parametrize("n_decode", [1, 5, 32])
def test_contraction_in_two_slices(hidden, mlp, n_decode):
    m = small_model(64, 8, 2, hidden=hidden, mlp=mlp, vocab=512)
    reqs = [W.RequestSpec(1, 7 + 3 * i) for i in range(n_decode)]
    w = W.build_workload("few", m, reqs, n_kv_pages=300, seed=300 + n_decode + hidden, std=0.02, resid_std=0.01)
    compare_layer(w, what=f"T={n_decode} H{hidden} I{mlp}")
