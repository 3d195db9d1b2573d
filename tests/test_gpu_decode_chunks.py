"""The decode kernel whose wavefronts take every W-th 32-key chunk, at the numbers of chunks where its loop can go wrong (none, one, two or
three for a wavefront, whole and cut short), whole contexts and parts, against the fp64 oracle.  Slots past the end of a
context hold NaN, which nothing may read."""
import pytest

import paper_2505_03780_amd as A
import workloads as W


@pytest.mark.gpu
@pytest.mark.parametrize("block", [16, 64, 1024])
@pytest.mark.parametrize("name", ["decode_bf16 d128 w8 split0", "decode_bf16 d128 w4 split0", "decode_bf16 d64 w8 split0", "decode_bf16 d64 w4 split0",
                                  "decode_f16 d128 w8 split0", "decode_f16 d64 w4 split0", "decode_bf16 d128 w8 split256", "decode_bf16 d128 w4 split512",
                                  "decode_f16 d64 w4 split256"])
def test_edges_of_the_chunk_loop(name, block):
    from attn_testlib import check_full

    names = [A.attn_instance_name(True, i) for i in range(A.attn_num_instances(True))]
    dtype, d, w, _ = name.split()
    D, step = int(d[1:]), 32 * int(w[1:])
    keys = [1, 16, 31, 32, 33, step - 32, step - 1, step, step + 1, step + 33, 2 * step - 1, 2 * step, 2 * step + 1, 3 * step + 15]
    wl = W.make_paged(300, "decode", [1] * len(keys), keys, 8, 2, D, block, sum(-(-n // block) for n in keys) + 2)
    for s, n in enumerate(keys):
        b = wl.block_table[s, (n - 1) // block]
        for x in (wl.k, wl.v):
            x[b, (n - 1) % block + 1:] = 0x7FC0
    if dtype == "decode_f16":
        wl = W.as_f16(wl)
    A.attn_force_instance(True, names.index(name))
    try:
        check_full(wl, True, name)
    finally:
        A.attn_force_instance(True, -1)
