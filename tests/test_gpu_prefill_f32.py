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


@pytest.mark.parametrize("Hq,Hkv,D", [(4, 4, 64), (4, 2, 128)])
@pytest.mark.parametrize("paged", [False, True])
def test_non_finite_values_reach_only_the_rows_that_see_them(Hq, Hkv, D, paged):
    """Infinities and NaN in V of one token (mid-tile, last of the sequence), causal: earlier rows stay what they are, later
    ones get what the sum over their visible keys gives."""
    lens, bad = [40, 33, 150], [(20, np.inf), (32, -np.inf), (130, np.nan)]
    if paged:
        wl = W.make_paged(103, "prefill", lens, lens, Hq, Hkv, D, 16, sum(-(-n // 16) for n in lens) + 1)
        wl = W.Workload("f32", "prefill", "f32", *(W.bf16_bits_to_f32(x) for x in (wl.q, wl.k, wl.v)), wl.query_start_loc, wl.seq_lens, wl.scale, True,
                        block_table=wl.block_table, block_size=16)
        at = lambda s, t: (int(wl.block_table[s, t // 16]), t % 16)
    else:
        wl = W.make_prefill_contiguous(103, lens, Hq, Hkv, D, dtype="f32")
        at = lambda s, t: (int(wl.query_start_loc[s]) + t,)
    dw = DeviceWorkload(wl)
    clean = to_host_f64(dw.run(False))
    for s, (t, x) in enumerate(bad):
        dw.v[at(s, t)][Hkv - 1, 5::16] = x
    got = to_host_f64(dw.run(False)).reshape(-1, Hkv, Hq // Hkv, D)
    want = clean.reshape(got.shape).copy()
    for s, (t, x) in enumerate(bad):
        q0 = int(wl.query_start_loc[s])
        want[q0 + t:q0 + lens[s], Hkv - 1, :, 5::16] = x
    assert np.array_equal(got, want, equal_nan=True)
