"""Keys that score -inf (a channel of K holds -inf, as a mask carried in the keys would) ahead of every finite score of a row: the
softmax runs over the rest, wherever its scores lie.  Every prefill and decode instance, against a softmax in 64 bits."""
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


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("D", [64, 128])
def test_decode_with_hidden_chunks(D, dtype):
    """Whole 32-key chunks of -inf, at the start of a context and inside it: the first chunk of one wavefront, of a part, of a run."""
    lens = [700, 320, 1000, 257]
    wl = W.make_paged(111, "decode", np.ones(len(lens), np.int32), lens, 8, 4, D, 16, sum(-(-n // 16) for n in lens) + 1, causal=False)
    if dtype == "f16":
        wl = W.as_f16(wl)
    dw = DeviceWorkload(wl)
    dw.q[..., 0] = 1.0
    dw.k[..., 0] = 0.0
    for s, n in enumerate(lens):
        for c in range(s % 2, n // 32, 2):  # every other chunk
            for j in range(2):
                dw.k[int(wl.block_table[s, 2 * c + j]), :, :, 0] = -torch.inf
    q, k, v = (to_host_f64(t) for t in (dw.q, dw.k, dw.v))
    ref = np.empty_like(q)
    for s, n in enumerate(lens):
        rows = wl.block_table[s, :-(-n // 16)]
        ks, vs = (t[rows].reshape(-1, 4, D)[:n] for t in (k, v))
        x = np.einsum("hgd,khd->hgk", q[s].reshape(4, 2, D), ks) * wl.scale
        p = np.exp(x - x.max(-1, keepdims=True))
        ref[s] = np.einsum("hgk,khd->hgd", p / p.sum(-1, keepdims=True), vs).reshape(8, D)
    done = 0
    try:
        for i in range(A.attn_num_instances(True)):
            A.attn_force_instance(True, i)
            if A.attn_selected_instance(dw.args(True), True) == i:
                assert_close(to_host_f64(dw.run(True)), ref, dtype, A.attn_instance_name(True, i))
                done += 1
    finally:
        A.attn_force_instance(True, -1)
    assert done >= 8
