"""The ring prefill kernel where its start and its end meet: sequences of one unit of 32 keys up to more than the ring holds, a
key to either side of every edge, by every instance.  Units past the last are not requested to fill the ring, so their slots hold
what an earlier workgroup left there (but at the end of a whole trip round the ring, which may repeat the last unit); here that is NaN, by a
call over NaN that reaches every compute unit twice."""
import numpy as np
import pytest
import torch

import paper_2505_03780_amd as A
import workloads as W
from attn_testlib import DeviceWorkload, assert_close, oracle_problem, to_host_f64

import oracle

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 160, 161, 192, 224, 225, 256, 257, 288, 289, 321]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("paged,causal,sign,Hkv", [(False, True, 1, 2), (True, True, -1, 2), (True, False, 1, 2), (True, True, 1, 1), (False, False, -1, 1)])
def test_every_instance_from_one_unit_to_a_full_ring(D, dtype, paged, causal, sign, Hkv):
    scale = sign / np.sqrt(D)
    if paged:
        # (the last: a wavefront whose one token is the tile's last one and sees whole units, next to others that do not)
        q_lens, kv_lens = [min(n, 40) for n in LENS] + [33, 65], LENS + [64, 128]
        wl = W.make_paged(95, "prefill", q_lens, kv_lens, 8, Hkv, D, 16, sum(-(-n // 16) for n in kv_lens) + 3, scale=scale, causal=causal)
    else:
        wl = W.make_prefill_contiguous(96, LENS, 8, Hkv, D, scale=scale, causal=causal)
    poison = W.make_prefill_contiguous(97, [256] * 64, 8, Hkv, D, scale=scale, causal=False)
    if dtype == "f16":
        wl, poison = W.as_f16(wl), W.as_f16(poison)
    dw, dp = DeviceWorkload(wl), DeviceWorkload(poison)
    for t in (dp.q, dp.k, dp.v):
        t.fill_(float("nan"))
    ref = oracle.attention(oracle_problem(wl))
    done = set()
    try:
        for i in range(A.attn_num_instances(False)):
            name = A.attn_instance_name(False, i)
            A.attn_force_instance(False, i)
            if "ring d%d" % D in name and A.attn_selected_instance(dw.args(False), False) == i:
                print(name, flush=True)
                assert torch.isnan(dp.run(False)).all()
                assert_close(to_host_f64(dw.run(False)), ref, dtype, name)  # tolerances of the element type, derived in attn_testlib
                done.add(name)
    finally:
        A.attn_force_instance(False, -1)
    # every ring instance of the type and head size whose heads per workgroup divide the group
    want = {n for n in (A.attn_instance_name(False, i) for i in range(A.attn_num_instances(False)))
            if n.startswith("prefill_%s_ring d%d " % (dtype, D)) and 8 // Hkv % int(n.split("hpw")[1].split()[0]) == 0}
    assert done == want and any("halves" in n for n in done)
