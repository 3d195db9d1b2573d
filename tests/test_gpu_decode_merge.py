"""The merge kernels of split decode at the edges of their blocks: as many parts as a block takes, one more, one less,
empty contexts among long ones, for the fixed-split and the token-balanced kernels, against the fp64 oracle."""
import numpy as np
import pytest

import paper_2505_03780_amd as A
import workloads as W
from attn_testlib import DeviceWorkload, assert_close, oracle_problem, to_host_f64

import oracle

pytestmark = pytest.mark.gpu


def _force(name):
    A.attn_force_instance(True, next(i for i in range(A.attn_num_instances(True)) if A.attn_instance_name(True, i) == name))


def _check(wl):
    """Sequences with keys against the oracle (tolerances of the element type), an empty context gives zeros."""
    got = to_host_f64(DeviceWorkload(wl).run(True))
    full = np.flatnonzero(wl.seq_lens)
    part = W.Workload(wl.name, "decode", wl.dtype, wl.q[full], wl.k, wl.v, np.arange(len(full) + 1, dtype=np.int32), wl.seq_lens[full],
                      wl.scale, True, block_table=wl.block_table[full], block_size=wl.block_size)
    assert_close(got[full], oracle.attention(oracle_problem(part)), wl.dtype)
    assert not got[wl.seq_lens == 0].any()


@pytest.mark.parametrize("G", [1, 4])  # one query head (an idle half of the merging wavefront), two pairs
@pytest.mark.parametrize("longest", [4, 5, 8, 9, 33])  # parts of 256 keys: blocks of 4, 8 and 32
def test_fixed_split(longest, G):
    lens = [256 * longest, 256 * longest - 255, 1, 0, 256, 257, 256 * 4 + 1]
    lens = [min(n, 256 * longest) for n in lens]
    wl = W.make_paged(95, "decode", np.ones(len(lens), np.int32), lens, 2 * G, 2, 128, 16, sum(-(-n // 16) for n in lens) + 1, causal=False)
    _force("decode_bf16 d128 w4 split256")
    try:
        _check(wl)
    finally:
        A.attn_force_instance(True, -1)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f16", 128), ("bf16", 64)])
@pytest.mark.parametrize("lens", [[3000, 0, 17, 1, 900], [20] * 40 + [4000] + [64] * 40, [40] * 300, [16000]])
def test_token_balanced(lens, dtype, D):
    """Few sequences for the runs (blocks of 32), as many (8, 4, with one sequence of far more parts than expected)."""
    wl = W.make_paged(96, "decode", np.ones(len(lens), np.int32), lens, 8, 2, D, 16, sum(-(-n // 16) for n in lens) + 1, causal=False)
    if dtype == "f16":
        wl = W.as_f16(wl)
    _force("decode_%s_balanced d%d w8 percu1" % (dtype, D))
    try:
        _check(wl)
    finally:
        A.attn_force_instance(True, -1)


@pytest.mark.parametrize("dtype,D,Hq,Hkv", [("bf16", 128, 8, 2), ("f16", 64, 3, 1)])
@pytest.mark.parametrize("lens", [
    [32 * 256 - 32 * 99] + [32] * 99,     # one chunk per run: the long context at the front, 157 parts
    [32] * 60 + [32 * 150] + [1] * 46,    # in the middle
    [0] * 30 + [32] * 200 + [32 * 17],    # at the end, 17 parts: one more than a wavefront of the ordinary merge takes on
    [32] * 200 + [32 * 16] + [0] * 30,    # 16 parts: the most that it does
    [32 * 40, 1, 32 * 40, 0, 32 * 40] + [20] * 95,  # several long ones next to each other
    [32 * 16 + 1] * 15 + [5] * 70,        # every helper's sequence is another one, 17 chunks each
    [32] * 5 + [32 * 32] + [0, 32],       # few sequences: 32 parts, the most that an ordinary merge takes on
    [32 * 33, 32], [32 * 100, 1, 32 * 99, 3], [32 * 256], [32 * 300, 5]])  # 33, two next to each other, a run each and more
def test_token_balanced_long_among_short(lens, dtype, D, Hq, Hkv):
    """Sequences of more parts than one wavefront merges, among many of one part."""
    wl = W.make_paged(98, "decode", np.ones(len(lens), np.int32), lens, Hq, Hkv, D, 16, sum(-(-n // 16) for n in lens) + 1, causal=False)
    if dtype == "f16":
        wl = W.as_f16(wl)
    _force("decode_%s_balanced d%d w8 percu1" % (dtype, D))
    try:
        _check(wl)
    finally:
        A.attn_force_instance(True, -1)


@pytest.mark.parametrize("skew,equal,name", [([32768] + [64] * 255, [192] * 256, "d64 w8 percu1"), ([8000] + [100] * 11, [758] * 12, "d128 w4 percu1")])
def test_merge_of_a_long_context_among_short_ones_is_not_serial(skew, equal, name):
    """One long context among short ones against equal contexts of as many keys in all: the kernels that walk the keys take the same
    time, and so must the merge, within a factor of two of the whole (with the long context's records walked block by block by one
    wavefront it was 2.6 and 2.4; it is 1.4 and 1.1)."""
    import torch

    def median_us(lens):
        wl = W.make_paged(99, "decode", np.ones(len(lens), np.int32), lens, 32, 8, int(name[1:4]), 16, sum(-(-n // 16) for n in lens) + 1, causal=False)
        dw = DeviceWorkload(wl)
        a = dw.args(True)
        assert "balanced" in A.attn_instance_name(True, A.attn_selected_instance(a, True))
        run = lambda: A.attn_decode_paged(None, None, None, None, None, None, None, max_kv_len=0, args=a)
        times = []
        for _ in range(30):
            e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
            for _ in range(3):
                run()
            e0.record()
            for _ in range(10):
                run()
            e1.record()
            e1.synchronize()
            times.append(100 * e0.elapsed_time(e1))
        return sorted(times)[15]

    A.attn_force_instance(True, next(i for i in range(A.attn_num_instances(True)) if A.attn_instance_name(True, i) == "decode_bf16_balanced " + name))
    try:
        skewed, even = median_us(skew), median_us(equal)
    finally:
        A.attn_force_instance(True, -1)
    print("skewed %.1f us, even %.1f us" % (skewed, even), flush=True)
    assert skewed <= 2.0 * even
