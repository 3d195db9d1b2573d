"""Keys that score -inf (a channel of K holds -inf, as a mask carried in the keys would) ahead of every finite score of a row: the
softmax runs over the rest, wherever its scores lie.  Every prefill instance, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2505_03780_amd as A
import workloads as W
from attn_testlib import DeviceWorkload, assert_close, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("level", [-20.0, -300.0])  # log2 of the later weights against a reference of 0: below fp16's normals, below fp32's
def test_scores_behind_a_hidden_head(D, level, dtype):
    n, hidden = 300, [0, 1, 32, 33, 64, 200]
    wl = W.make_prefill_contiguous(110, [n] * len(hidden), 4, 1, D, causal=False)
    if dtype == "f16":
        wl = W.as_f16(wl)
    dw = DeviceWorkload(wl)
    dw.q[..., 0] = 1.0
    dw.k[..., 0] = level / (wl.scale * 1.4426950408889634)
    for s, h in enumerate(hidden):
        dw.k[s * n:s * n + h, :, 0] = -torch.inf
    q, k, v = (to_host_f64(t) for t in (dw.q, dw.k, dw.v))
    ref = np.empty_like(q)
    for s in range(len(hidden)):
        rows = slice(s * n, (s + 1) * n)
        x = np.einsum("thd,kd->thk", q[rows], k[rows, 0]) * wl.scale
        p = np.exp(x - x.max(-1, keepdims=True))
        ref[rows] = np.einsum("thk,kd->thd", p / p.sum(-1, keepdims=True), v[rows, 0])
    done = 0
    try:
        for i in range(A.attn_num_instances(False)):
            A.attn_force_instance(False, i)
            if A.attn_selected_instance(dw.args(False), False) == i:
                assert_close(to_host_f64(dw.run(False)), ref, dtype, A.attn_instance_name(False, i))
                done += 1
    finally:
        A.attn_force_instance(False, -1)
    assert done >= 5
