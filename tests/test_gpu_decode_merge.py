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
