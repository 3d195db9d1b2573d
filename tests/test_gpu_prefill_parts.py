"""Prefill whose keys are cut into parts over workgroups (a call that brings scratch memory), by the key-split and by the ring
kernel: results at the edges of tiles and parts against the fp64 oracle, the calls that take a workspace, and those that must do without."""
import numpy as np
import pytest

import paper_2505_03780_amd as A
import workloads as W
from test_host_api import _args, _paged
from test_prefill_split import _instance, _packed


def test_calls_that_take_a_workspace():
    A.attn_clear_cache()
    A.attn_force_instance(False, -1)
    turn = dict(num_seqs=2, total_q=12, block_table_stride=2048, max_q_len=8)  # 16 tiles of 8 tokens
    a = _paged(max_kv_len=8000, **turn)
    assert A.attn_prefill_scratch_bytes(a) == 16 * 16 * 32 * 130 * 4  # 16 parts of two steps of 256 keys in one round
    assert A.attn_workspace_bytes(a, False) == 0  # needed: none
    assert A.attn_prefill_scratch_bytes(_paged(max_kv_len=1024, **turn)) == 0  # nothing to gain
    # new tokens enough for 128-row tiles: the ring kernel in parts, whether its unsplit form was the choice or not
    turns = dict(num_seqs=3, total_q=130, block_table_stride=2048, max_q_len=70)
    assert A.attn_prefill_scratch_bytes(_paged(max_kv_len=7948, **turns)) == 72 * 8 * 128 * 130 * 4
    assert A.attn_prefill_scratch_bytes(_paged(num_seqs=1, total_q=1000, block_table_stride=2048, max_q_len=1000, max_kv_len=8192)) > 0
    # enough tiles
    assert A.attn_prefill_scratch_bytes(_paged(max_kv_len=8000, num_seqs=16, total_q=8192, max_q_len=512, block_table_stride=2048)) == 0
    one = _paged(num_seqs=1, total_q=1, block_table_stride=1 << 16, max_q_len=1, max_kv_len=1 << 20)
    assert A.attn_prefill_scratch_bytes(one) == 8 * 32 * 32 * 130 * 4  # one round
    a.struct_bytes += 8
    assert A.attn_prefill_scratch_bytes(a) == 0
    # a bound that says nothing, as packed keys may have, is a very long context
    free = lambda n: A.attn_prefill_scratch_bytes(_args(num_seqs=1, total_q=8, max_q_len=8, max_kv_len=n))
    assert free(2 ** 31 - 1) == free(2 ** 30) > 0
    # no more than four records of 128 rows per compute unit
    assert A.attn_prefill_scratch_bytes(_paged(num_seqs=16, total_q=144, max_q_len=128, max_kv_len=3000, block_table_stride=256)) <= 1024 * 128 * 130 * 4


def _ring(dtype, D, Hq, Hkv):
    g = Hq // Hkv
    name = "prefill_%s_ring d%d qb1 w4 hpw%d slots4 pf4 seqmajor" % (dtype, D, 4 if g % 4 == 0 else 2 if g % 2 == 0 else 1)
    return next(i for i in range(A.attn_num_instances(False)) if A.attn_instance_name(False, i) == name)


SHAPES = [  # kernel, Hq, Hkv, D, block (0: packed), new tokens, keys; more than 1024 keys are cut (ring: 2048 or more)
    ("split", 8, 2, 128, 16, [9, 1, 8], [1025, 1300, 40]),           # parts of 256; a sequence shorter than a part
    ("split", 8, 2, 64, 0, [9, 1, 33], [2049, 1792, 257]),
    ("split", 4, 4, 128, 64, [33, 2], [3000, 2999]),                 # a second tile of one row
    ("split", 6, 2, 128, 0, [5, 0, 12], [2305, 64, 2304]),           # one head a tile, an empty query; a part of one key
    ("split", 64, 1, 128, 16, [1, 2], [5000, 17]),                   # two sub-groups of 32 heads
    ("split", 1, 1, 64, 512, [1700], [3700]),                        # a late part that the early tiles do not see at all
    ("ring", 8, 2, 128, 16, [33, 1, 32], [2048, 2305, 40]),          # 4 heads x 32 tokens a tile; a part of one key; no parts
    ("ring", 8, 2, 64, 0, [65, 31, 5], [4097, 2559, 257]),
    ("ring", 4, 2, 128, 1024, [70, 1], [3000, 4095]),                # 2 heads a tile; parts that start inside a cache block
    ("ring", 3, 3, 128, 0, [129, 0, 12], [2100, 64, 6000]),          # one head a tile, an empty query
    ("ring", 16, 4, 64, 128, [40, 3], [7000, 2048]),
    ("ring", 1, 1, 128, 16, [3000], [3100]),                         # late parts that the early tiles do not see, or not fully
]


def _run(dw, ws, nbytes=None):
    import torch

    ws = ws.view(torch.uint8)
    dw.out.fill_(float("nan"))
    A.attn_prefill_varlen(None, None, None, None, None, None, None, max_q_len=0, max_kv_len=0, args=dw.args(False), workspace=ws[:nbytes])
    return dw.out


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal,scale", [(True, 1.0), (False, -6.0)])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
def test_parts_against_the_oracle(shape, causal, scale, dtype):
    import torch
    from attn_testlib import TOL, DeviceWorkload, oracle_problem, to_host_f64

    import oracle

    kernel, Hq, Hkv, D, block, new, keys = SHAPES[shape]
    bs = block or 16
    wl = W.make_paged(170 + shape, "prefill", new, keys, Hq, Hkv, D, bs, sum(-(-n // bs) for n in keys) + 3, scale=scale / np.sqrt(D), causal=causal)
    if block:
        for s, n in enumerate(keys):  # slots past the end of a sequence hold NaN: nothing may read them
            b = wl.block_table[s, (n - 1) // block]
            wl.k[b, (n - 1) % block + 1:] = 0x7FC0
            wl.v[b, (n - 1) % block + 1:] = 0x7FC0
    else:
        wl = _packed(wl)
    if dtype == "f16":
        wl = W.as_f16(wl)
    dw = DeviceWorkload(wl)
    ref = oracle.attention(oracle_problem(wl))
    A.attn_force_instance(False, _instance(dtype, D) if kernel == "split" else _ring(dtype, D, Hq, Hkv))
    try:
        need = A.attn_prefill_scratch_bytes(dw.args(False))
        assert need > 0
        ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")  # needs no initialisation
        split = to_host_f64(_run(dw, ws))
        again = to_host_f64(_run(dw, ws))
        whole = to_host_f64(_run(dw, ws, need - 1))  # too small: ignored
        assert np.array_equal(whole, to_host_f64(dw.run(False)))
    finally:
        A.attn_force_instance(False, -1)
    assert np.array_equal(split, again)
    # tolerances of the element type, derived in attn_testlib
    for got in (split, whole):
        assert np.abs(got - ref).max() <= TOL[dtype][0] and np.linalg.norm(got - ref) <= TOL[dtype][1] * np.linalg.norm(ref)


@pytest.mark.gpu
@pytest.mark.parametrize("kernel,D", [("split", 128), ("split", 64), ("ring", 128), ("ring", 64)])
def test_layouts_in_parts_give_the_same_bits(kernel, D):
    """Queries, outputs and caches with other strides, and packed keys, through the records and the merge."""
    import torch
    from attn_testlib import DeviceWorkload, to_host_f64

    paged = W.make_paged(184, "prefill", [40, 9], [4100, 2333], 8, 2, D, 16, 420)
    dw = DeviceWorkload(paged)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    A.attn_force_instance(False, _instance("bf16", D) if kernel == "split" else _ring("bf16", D, 8, 2))
    try:
        assert A.attn_prefill_parts_instance(dw.args(False))[1] > 1
        ref = to_host_f64(_run(dw, ws))
        assert np.array_equal(to_host_f64(_run(DeviceWorkload(_packed(paged)), ws)), ref)
        q, out, k, v = dw.q, dw.out, dw.k, dw.v
        for name, t in (("q", q), ("out", out)):
            wide = torch.zeros(49, 8, 2 * D + 8, dtype=torch.bfloat16, device="cuda")
            wide[:, :, D:2 * D] = t
            setattr(dw, name, wide[:, :, D:2 * D])
        assert np.array_equal(to_host_f64(_run(dw, ws)), ref)
        dw.k, dw.v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (k, v))  # heads outside the slots of a block
        assert np.array_equal(to_host_f64(_run(dw, ws)), ref)
    finally:
        A.attn_force_instance(False, -1)


@pytest.mark.gpu
@pytest.mark.parametrize("tensor,value", [("v", 0x7F80), ("v", 0xFF80), ("v", 0x7FC0), ("k", 0x7F80), ("k", 0x7FC0)])
@pytest.mark.parametrize("kernel,D,new,keys", [("split", 128, 9, 3000), ("split", 64, 9, 2700), ("ring", 128, 33, 3000), ("ring", 64, 40, 4200)])
def test_infinities_and_nan_through_the_merge(kernel, D, new, keys, tensor, value):
    """A non-finite key or value in the first, the last or several parts reaches the outputs that it reaches without parts, as the
    same infinity or as NaN: where the number of parts is no multiple of the merge's eight, too."""
    import torch
    from attn_testlib import DeviceWorkload, to_host_f64

    for at in ([keys - new - 3], [5], [5, keys - new - 3], [keys - 3]):  # (the last: seen by some queries only)
        wl = W.make_paged(175, "prefill", [new], [keys], 8, 2, D, 16, -(-keys // 16) + 3)
        for key in at:
            getattr(wl, tensor)[wl.block_table[0, key // 16], key % 16, 0, 7] = value
        dw = DeviceWorkload(wl)
        A.attn_force_instance(False, _instance("bf16", D) if kernel == "split" else _ring("bf16", D, 8, 2))
        try:
            need = A.attn_prefill_scratch_bytes(dw.args(False))
            rows = 32 if kernel == "split" else 128
            tiles = 2 * -(-new // (rows // 4))
            parts = need // (tiles * rows * (D + 2) * 4)
            assert parts > 1 and parts % 8 != 0
            split = to_host_f64(_run(dw, torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")))
            whole = to_host_f64(dw.run(False))
        finally:
            A.attn_force_instance(False, -1)
        assert not np.isfinite(whole[-1]).all() and np.isfinite(whole[:, 4:]).all()  # (the other KV head)
        if (tensor, value) == ("v", 0x7F80):
            assert (whole[-1, :4, 7] == np.inf).all()
        for pattern in (np.isnan, np.isposinf, np.isneginf):
            differ = int((pattern(split) != pattern(whole)).sum())
            assert differ == 0, (at, pattern.__name__)


def test_a_tuned_winner_stands(tmp_path):
    """Only the built-in choice gives way to parts by the library's models; a winner was measured."""
    A.attn_clear_cache()
    A.attn_force_instance(False, -1)
    a = _paged(num_seqs=3, total_q=130, block_table_stride=2048, max_q_len=70, max_kv_len=7948)
    need = A.attn_prefill_scratch_bytes(a)
    assert need > 0
    built_in = A.attn_selected_instance(a, False)
    for winner in (built_in, _instance("bf16", 128), _ring("bf16", 128, 32, 8)):
        f = tmp_path / "c.txt"
        f.write_text("attn-tune-cache-v1\n%s\tprefill|bf16|d128|hq32|hkv8|paged|bs16|c1|B2|q7|kv13\t%s\t1.0\n" % (A.attn_environment_key(), A.attn_instance_name(False, winner)))
        assert A.attn_load_cache(str(f)) == 0
        assert A.attn_selected_instance(a, False) == winner and A.attn_prefill_scratch_bytes(a) == 0
    A.attn_clear_cache()
    assert A.attn_selected_instance(a, False) == built_in and A.attn_prefill_scratch_bytes(a) == need


def test_the_plan_is_reported():
    """The instance and the parts that a call with scratch memory launches; attn_selected_instance speaks of the call without."""
    import os
    import subprocess
    import sys

    A.attn_clear_cache()
    A.attn_force_instance(False, -1)
    a = _paged(num_seqs=3, total_q=130, block_table_stride=2048, max_q_len=70, max_kv_len=7948)
    selected, (planned, parts) = A.attn_selected_instance(a, False), A.attn_prefill_parts_instance(a)
    assert "keysplit" in A.attn_instance_name(False, selected) and planned == _ring("bf16", 128, 32, 8)
    assert A.attn_prefill_scratch_bytes(a) == 72 * parts * 128 * 130 * 4
    short = _paged(num_seqs=3, total_q=130, block_table_stride=2048, max_q_len=70, max_kv_len=1000)
    assert A.attn_prefill_parts_instance(short) == (A.attn_selected_instance(short, False), 1)
    with pytest.raises(A.AttnError):
        A.attn_prefill_parts_instance(_paged(head_dim=80))
    here = os.path.dirname(os.path.abspath(__file__))
    code = ("import sys; sys.path[:0] = [%r, %r]\nimport test_host_api as T, paper_2505_03780_amd as A\n"
            "A.attn_prefill_scratch_bytes(T._paged(num_seqs=3, total_q=130, block_table_stride=2048, max_q_len=70, max_kv_len=7948))\n" % (os.path.dirname(here), here))
    env = dict(os.environ, ATTN_LOG="1")
    env.pop("ATTN_FORCE_INSTANCE", None)
    log = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=100).stderr
    assert "with scratch memory -> %s in %d parts" % (A.attn_instance_name(False, planned), parts) in log


def test_refusals_are_those_of_the_call_without_scratch_memory():
    args = dict(num_seqs=2, total_q=12, block_table_stride=2048, max_q_len=8, max_kv_len=8000)
    for change in (dict(dtype=7), dict(num_kv_heads=3), dict(head_dim=80), dict(block_size=24), dict(q=0), dict(seq_lens=0), dict(k=0x100008)):
        a = _paged(**dict(args, **change))
        status = []
        for call in (lambda: A.load_library().attn_prefill_varlen(a, None), lambda: A.load_library().attn_prefill_varlen_parts(a, 0x100000, 1 << 30, None)):
            status.append(call())
        assert status[0] == status[1] < 0, change


@pytest.mark.gpu
def test_a_workspace_in_the_struct_is_not_touched():
    """One workspace pointer in the structs of decode and prefill calls that overlap is safe: prefill ignores it."""
    import torch
    from attn_testlib import DeviceWorkload

    dw = DeviceWorkload(W.make_paged(181, "prefill", [5, 3], [4000, 3000], 8, 2, 128, 16, 450))
    whole = dw.run(False).clone()
    a = dw.args(False)
    need = A.attn_prefill_scratch_bytes(a)
    assert need > 0
    ws = torch.full((2 * need,), 7, dtype=torch.uint8, device="cuda")
    a.workspace, a.workspace_bytes = ws.data_ptr(), ws.nbytes
    dw.out.fill_(float("nan"))
    A.attn_prefill_varlen(None, None, None, None, None, None, None, max_q_len=0, max_kv_len=0, args=a)
    assert torch.equal(dw.out, whole) and bool((ws == 7).all())


@pytest.mark.gpu
def test_a_captured_call_with_a_workspace_gives_the_eager_bits():
    import torch
    from attn_testlib import DeviceWorkload

    dw = DeviceWorkload(W.make_paged(182, "prefill", [5, 3], [4000, 3000], 8, 2, 128, 16, 450))
    ws = torch.empty(A.attn_prefill_scratch_bytes(dw.args(False)), dtype=torch.uint8, device="cuda")
    run = lambda **kw: A.attn_prefill_varlen(dw.q, dw.k, dw.v, dw.out, dw.qsl, dw.seq_lens, dw.wl.scale, max_q_len=dw.max_q, max_kv_len=dw.max_kv,
                                             block_table=dw.bt, **kw)
    run()
    eager = dw.out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(workspace=ws)
    for _ in range(3):
        dw.out.fill_(float("nan"))
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dw.out, eager)


@pytest.mark.gpu
def test_tensor_call_takes_and_leaves_the_workspace():
    """A call with tensors gives the bits of a call with a workspace, on a side stream too; under capture it does without."""
    import torch
    from attn_testlib import DeviceWorkload

    dw = DeviceWorkload(W.make_paged(180, "prefill", [5, 3], [4000, 3000], 8, 2, 128, 16, 450))
    call = dict(max_q_len=dw.max_q, max_kv_len=dw.max_kv, causal=True, block_table=dw.bt)
    run = lambda **kw: A.attn_prefill_varlen(dw.q, dw.k, dw.v, dw.out, dw.qsl, dw.seq_lens, dw.wl.scale, **call, **kw)
    need = A.attn_prefill_scratch_bytes(dw.args(False))
    assert need > 0
    split = _run(dw, torch.empty(need, dtype=torch.uint8, device="cuda")).clone()
    whole = dw.run(False).clone()
    assert not torch.equal(split, whole)  # (other rounding: the two are told apart below)
    dw.out.fill_(float("nan"))
    run()
    assert torch.equal(dw.out, split)
    side = torch.cuda.Stream()
    dw.out.fill_(float("nan"))
    torch.cuda.synchronize()
    run(stream=side)
    torch.cuda.synchronize()
    assert torch.equal(dw.out, split)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for _ in range(3):
        dw.out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dw.out, whole)


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["handle", "fake tensors", "another capture", "short memory"])
def test_calls_that_taking_scratch_memory_must_not_disturb(how):
    """What a call served before it took scratch memory it serves still: on a stream object that only has a handle, under a mode that
    makes new tensors fake ones, beside another stream's capture, and with no memory left (which must not cost the
    allocator's cache on every call)."""
    import threading
    import types

    import torch
    from attn_testlib import DeviceWorkload

    dw = DeviceWorkload(W.make_paged(183, "prefill", [5, 3], [4000, 3000], 8, 2, 128, 16, 450))
    assert A.attn_prefill_scratch_bytes(dw.args(False)) > 0
    run = lambda **kw: A.attn_prefill_varlen(dw.q, dw.k, dw.v, dw.out, dw.qsl, dw.seq_lens, dw.wl.scale, max_q_len=dw.max_q, max_kv_len=dw.max_kv,
                                             block_table=dw.bt, **kw)
    side = torch.cuda.Stream()
    whole = dw.run(False).clone()
    run(stream=side)
    torch.cuda.synchronize()
    split = dw.out.clone()
    assert not torch.equal(split, whole)
    dw.out.fill_(float("nan"))
    torch.cuda.synchronize()
    if how == "handle":
        run(stream=types.SimpleNamespace(cuda_stream=side.cuda_stream))
        torch.cuda.synchronize()
        assert torch.equal(dw.out, whole)
    elif how == "fake tensors":
        from torch._subclasses.fake_tensor import FakeTensorMode

        with FakeTensorMode():
            run()
        torch.cuda.synchronize()
        assert torch.equal(dw.out, split)
    elif how == "another capture":
        x, graph = torch.zeros(64, device="cuda"), torch.cuda.CUDAGraph()
        torch.cuda.empty_cache()  # the scratch memory has to come from the device
        with torch.cuda.graph(graph):
            x += 1
            run(stream=side)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dw.out, split) and bool((x == 1).all())
    else:
        failed = []

        def calls():  # (in a thread of its own: it does without for a while)
            torch.cuda.empty_cache()
            before = torch.cuda.memory_stats()["num_alloc_retries"]
            torch.cuda.set_per_process_memory_fraction(1e-6)
            try:
                for _ in range(5):
                    run(stream=side)
            finally:
                torch.cuda.set_per_process_memory_fraction(1.0)
            failed.append(torch.cuda.memory_stats()["num_alloc_retries"] - before)

        t = threading.Thread(target=calls)
        t.start()
        t.join()
        torch.cuda.synchronize()
        assert torch.equal(dw.out, whole) and failed[0] <= 1
