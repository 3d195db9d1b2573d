"""The fp32 prefill kernel at the edges of its tiles (16 rows of heads x tokens, 16-key chunks dealt over eight wavefronts),
with strides and addresses that are only dword aligned, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_03780_amd as A
import workloads as W
from attn_testlib import DeviceWorkload, assert_close, check_full, oracle_problem, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,D", [(4, 4, 64), (8, 2, 128), (3, 1, 64), (32, 1, 64), (2, 1, 128)])
@pytest.mark.parametrize("causal,scale", [(True, 1.0), (False, -6.0)])
def test_tile_and_chunk_edges(Hq, Hkv, D, causal, scale):
    lens = [1, 15, 16, 17, 0, 127, 128, 129, 300]  # chunks: one, eight exactly, nine; rows: a tile less one, exactly, one more
    check_full(W.make_prefill_contiguous(101, lens, Hq, Hkv, D, dtype="f32", scale=scale / np.sqrt(float(D)), causal=causal))


def test_dword_aligned_views():
    """No stride or address of an fp32 call has to be a multiple of 16 bytes."""
    wl = W.make_prefill_contiguous(102, [33, 70], 4, 2, 64, dtype="f32")
    ref = oracle.attention(oracle_problem(wl))
    dw = DeviceWorkload(wl)
    aligned = to_host_f64(dw.run(False))

    def view(t):  # rows of 67 floats, first element one float into the buffer
        buf = torch.full((t.shape[0] * t.shape[1] * 67 + 1,), float("nan"), device="cuda")
        v = buf[1:].view(t.shape[0], t.shape[1], 67)[:, :, :64]
        v.copy_(t)
        return v

    dw.q, dw.k, dw.v, dw.out = view(dw.q), view(dw.k), view(dw.v), view(dw.out)
    got = to_host_f64(dw.run(False))
    assert np.array_equal(got, aligned)
    assert_close(got, ref, "f32")
