"""The ring prefill kernel at head size 128, every instance: a peaked softmax, whose reference moves inside the loop, keys visible
to every query, a sign that moves into Q, over lengths that reach each of its loops (the pass round an eight- or four-slot
ring, the plain units left over, masked units, one unit), against the fp64 oracle.  The built-in choice gives calls this small
to the key-split kernel, so the instances are forced."""
import numpy as np
import pytest

import paper_2505_03780_amd as A
import workloads as W
from attn_testlib import DeviceWorkload, assert_close, oracle_problem, to_host_f64

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("Hq,Hkv,paged,causal,scale", [(8, 1, False, True, 6.0), (8, 2, False, False, 1.0), (4, 2, True, True, -5.0), (8, 1, True, False, 4.0)])
def test_every_d128_ring_instance(Hq, Hkv, paged, causal, scale, dtype):
    scale /= np.sqrt(128.0)
    if paged:  # chunks behind a prefix: rows whose first masked unit lies anywhere in the ring
        q_lens, kv_lens, bs = [1, 70, 64, 129, 33], [289, 70, 64 + 512, 129 + 640, 33 + 95], 32
        wl = W.make_paged(93, "prefill", q_lens, kv_lens, Hq, Hkv, 128, bs, sum(-(-n // bs) for n in kv_lens) + 2, scale=scale, causal=causal)
        for s, n in enumerate(kv_lens):  # unused slots hold NaN: nothing may use them
            b = wl.block_table[s, (n - 1) // bs]
            wl.k[b, (n - 1) % bs + 1:] = 0x7FC0
            wl.v[b, (n - 1) % bs + 1:] = 0x7FC0
    else:
        wl = W.make_prefill_contiguous(94, [1, 32, 33, 300, 0, 640, 1000], Hq, Hkv, 128, scale=scale, causal=causal)
    if dtype == "f16":
        wl = W.as_f16(wl)
    dw = DeviceWorkload(wl)
    ref = oracle.attention(oracle_problem(wl))
    done = set()
    try:
        for i in range(A.attn_num_instances(False)):
            name = A.attn_instance_name(False, i)
            A.attn_force_instance(False, i)
            if "ring d128" in name and A.attn_selected_instance(dw.args(False), False) == i:
                print(name, flush=True)
                assert_close(to_host_f64(dw.run(False)), ref, dtype, name)  # tolerances of the element type, derived in attn_testlib
                done.add(name)
    finally:
        A.attn_force_instance(False, -1)
    # every ring instance of the type whose heads per workgroup divide the group
    want = {n for n in (A.attn_instance_name(False, i) for i in range(A.attn_num_instances(False)))
            if n.startswith("prefill_%s_ring d128" % dtype) and (Hq // Hkv) % int(n.split("hpw")[1].split()[0]) == 0}
    assert done == want and len(done) >= 6
