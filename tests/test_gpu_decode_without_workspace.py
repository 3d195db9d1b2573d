"""Decode calls that the library serves without a workspace (whole contexts, one workgroup per KV head) although with one it
would split them, and calls that it refuses without one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_03780_amd as A
import workloads as W
from attn_testlib import DeviceWorkload, assert_close, oracle_problem, to_host_f64

pytestmark = pytest.mark.gpu


def _call(B, bound, Hq, Hkv, D, dtype):
    """B contexts of a few hundred keys under a host bound of `bound` keys (the choice goes by the bound)."""
    lens = np.random.default_rng(B).integers(1, min(bound, 300), size=B, endpoint=True)
    lens[-1] = min(bound, 1000)
    wl = W.make_paged(120, "decode", np.ones(B, np.int32), lens, Hq, Hkv, D, 16, int(sum(-(-n // 16) for n in lens)) + 1, table_width=-(-bound // 16),
                      causal=False)
    return DeviceWorkload(W.as_f16(wl) if dtype == "f16" else wl), W.as_f16(wl) if dtype == "f16" else wl


def _decode(dw, bound, workspace):
    dw.out.fill_(float("nan"))
    A.attn_decode_paged(dw.q, dw.k, dw.v, dw.out, dw.bt, dw.seq_lens, dw.wl.scale, max_kv_len=bound, workspace=workspace)
    torch.cuda.synchronize()
    return to_host_f64(dw.out)


@pytest.mark.parametrize("B,bound,Hq,Hkv,D,dtype", [(6, 6000, 32, 8, 64, "bf16"), (1, 1000, 32, 8, 64, "bf16"), (600, 3000, 8, 2, 128, "bf16"),
                                                    (142, 15000, 8, 2, 64, "bf16"), (70, 26000, 8, 2, 128, "f16")])
@pytest.mark.parametrize("given", [None, 64])  # nothing, a few bytes
def test_served(B, bound, Hq, Hkv, D, dtype, given):
    dw, wl = _call(B, bound, Hq, Hkv, D, dtype)
    a = A.make_args(dw.q, dw.k, dw.v, dw.out, dw.seq_lens, wl.scale, max_q_len=1, max_kv_len=bound, block_table=dw.bt, is_decode=True)
    assert "split0" not in A.attn_instance_name(True, A.attn_selected_instance(a, True))  # what a call with a workspace takes
    got = _decode(dw, bound, given and torch.empty(given, dtype=torch.uint8, device="cuda"))
    assert_close(got, oracle.attention(oracle_problem(wl)), dtype)


@pytest.mark.parametrize("B,bound,Hq,Hkv,D,dtype", [(4, 4096, 32, 8, 128, "bf16"), (64, 4096, 32, 8, 128, "bf16"), (64, 4096, 32, 8, 64, "f16")])
def test_refused(B, bound, Hq, Hkv, D, dtype):
    dw, _ = _call(B, bound, Hq, Hkv, D, dtype)
    for workspace in (None, torch.empty(64, dtype=torch.uint8, device="cuda")):
        with pytest.raises(A.AttnError):
            _decode(dw, bound, workspace)
    assert bool(torch.isnan(dw.out).all())


def test_a_forced_instance_is_not_replaced():
    dw, _ = _call(6, 6000, 32, 8, 64, "bf16")
    A.attn_force_instance(True, next(i for i in range(A.attn_num_instances(True)) if A.attn_instance_name(True, i) == "decode_bf16 d64 w4 split512"))
    try:
        with pytest.raises(A.AttnError):
            _decode(dw, 6000, None)
    finally:
        A.attn_force_instance(True, -1)
