"""The prefill kernel whose wavefronts split the keys (few query rows over many keys): its results at the edges of its
tiles against the fp64 oracle, and the rule that chooses it."""
import numpy as np
import pytest

import paper_2505_03780_amd as A
import workloads as W
from test_host_api import _args, _paged


def _instance(dtype, D):
    name = "prefill_%s_keysplit d%d w8" % (dtype, D)
    return next(i for i in range(A.attn_num_instances(False)) if A.attn_instance_name(False, i) == name)


def test_rule_on_the_host():
    A.attn_clear_cache()
    A.attn_force_instance(False, -1)
    name = lambda a: A.attn_instance_name(False, A.attn_selected_instance(a, False))
    turn = dict(num_seqs=2, total_q=60, block_table_stride=1024, max_q_len=32)  # 2 x 4 tiles of 8 tokens x 8 KV heads
    assert name(_paged(max_kv_len=8000, **turn)) == "prefill_bf16_keysplit d128 w8"
    assert name(_paged(max_kv_len=8000, dtype=A.ATTN_F16, **turn)) == "prefill_f16_keysplit d128 w8"
    assert name(_paged(max_kv_len=160, **turn)) == "prefill_bf16_keysplit d128 w8"
    assert "ring" in name(_paged(max_kv_len=159, **turn))  # nothing to split
    # one workgroup of 8 tokens per compute unit and KV head: 32 x 8 tokens over 8 heads fill 256 units
    assert "keysplit" in name(_args(num_seqs=1, total_q=256, max_q_len=256, max_kv_len=256))
    assert "ring" in name(_args(num_seqs=1, total_q=257, max_q_len=257, max_kv_len=257))
    many = dict(num_seqs=8, total_q=512, max_q_len=64, block_table_stride=1024)  # 512 workgroups
    assert "keysplit" in name(_paged(max_kv_len=1537, **many)) and "ring" in name(_paged(max_kv_len=1536, **many))
    small = dict(many, head_dim=64)
    assert name(_paged(max_kv_len=1025, **small)) == "prefill_bf16_keysplit d64 w8" and "ring d64" in name(_paged(max_kv_len=1024, **small))
    assert "ring" in name(_paged(max_kv_len=9000, **dict(many, max_q_len=65)))
    # head groups that are no power of two split into the largest power of two that divides them
    assert "keysplit" in name(_paged(max_kv_len=8000, num_q_heads=24, **turn))


SHAPES = [  # Hq, Hkv, D, block (0: packed), new tokens, keys
    (8, 2, 128, 0, [1, 7, 8, 9, 33], [1, 7, 8, 9, 33]),          # no prefix
    (2, 2, 64, 0, [1, 65], [1, 65]),
    (8, 2, 128, 0, [1, 7, 8, 9, 33], [1, 31, 32, 33, 257]),      # 4 heads x 8 tokens a tile; chunk edges
    (8, 2, 128, 0, [5, 1, 9, 8], [255, 256, 300, 520]),          # a wavefront's second and third chunk
    (4, 4, 128, 16, [31, 32, 33, 1], [255, 256, 257, 1030]),     # 1 head x 32 tokens; eight chunks exactly, one less, one more
    (6, 2, 128, 32, [5, 2, 70], [5, 700, 300]),                  # group of 3: one head a tile, three sub-groups
    (64, 1, 128, 16, [1, 2], [600, 17]),                         # group of 64: 32 heads x 1 token, two sub-groups
    (16, 2, 64, 128, [3, 4, 5, 0], [3, 290, 2000, 64]),          # D = 64, 8 heads x 4 tokens, an empty query
    (2, 2, 64, 0, [1, 65, 2, 31, 33], [40, 65, 255, 257, 520]),
]


def _packed(wl):
    """The keys of a paged workload laid end to end."""
    rows = [np.concatenate([x[wl.block_table[s, :-(-int(n) // wl.block_size)]].reshape(-1, *x.shape[2:])[:n] for s, n in enumerate(wl.seq_lens)])
            for x in (wl.k, wl.v)]
    start = np.concatenate([[0], np.cumsum(wl.seq_lens)]).astype(np.int32)
    return W.Workload("packed", wl.kind, wl.dtype, wl.q, rows[0], rows[1], wl.query_start_loc, wl.seq_lens, wl.scale, wl.causal, kv_start_loc=start)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal,scale", [(True, 1.0), (False, -6.0)])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_edges_against_the_oracle(shape, causal, scale, dtype):
    from attn_testlib import check_full

    Hq, Hkv, D, block, new, keys = SHAPES[shape]
    scale /= np.sqrt(float(D))  # (-6: a peaked softmax, and the sign moves into Q)
    bs = block or 16
    wl = W.make_paged(70 + shape, "prefill", new, keys, Hq, Hkv, D, bs, sum(-(-n // bs) for n in keys) + 3, scale=scale, causal=causal)
    if block:
        for s, n in enumerate(keys):  # slots past the end of a sequence hold NaN: nothing may read them
            b = wl.block_table[s, (n - 1) // block]
            wl.k[b, (n - 1) % block + 1:] = 0x7FC0
            wl.v[b, (n - 1) % block + 1:] = 0x7FC0
    else:
        wl = _packed(wl)
    if dtype == "f16":
        wl = W.as_f16(wl)
    A.attn_force_instance(False, _instance(dtype, D))
    try:
        check_full(wl, False)  # tolerances of the element type, derived in attn_testlib
    finally:
        A.attn_force_instance(False, -1)


@pytest.mark.gpu
def test_layouts_give_the_same_bits():
    """Packed and paged keys, and a query view with other strides, take the same arithmetic."""
    import torch
    from attn_testlib import DeviceWorkload, to_host_f64

    q_lens, kv_lens = [40, 9], [900, 333]
    paged = W.make_paged(81, "prefill", q_lens, kv_lens, 8, 2, 128, 16, 90)
    dw = DeviceWorkload(paged)
    A.attn_force_instance(False, _instance("bf16", 128))
    try:
        ref = to_host_f64(dw.run(False))
        packed = _packed(paged)
        assert np.array_equal(to_host_f64(DeviceWorkload(packed).run(False)), ref)
        wide = torch.zeros(49, 8, 264, dtype=torch.bfloat16, device="cuda")
        wide[:, :, 128:256] = dw.q
        dw.q = wide[:, :, 128:256]
        assert np.array_equal(to_host_f64(dw.run(False)), ref)
    finally:
        A.attn_force_instance(False, -1)
