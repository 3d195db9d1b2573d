"""The native marshalling of the tensor calls against the general Python path: the same struct for every plain call, and None (the
general path decides) for everything else.  The structs hold CPU pointers and nothing is called with them, but for the GPU test."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2505_03780_amd as A
from paper_2505_03780_amd import binding as B
from test_binding_args import _case, _NoStream

B._dtype_codes()  # loads the extension
F = B._fast


def _pack(c):
    return F.attn(-1, *c.values())


@pytest.mark.parametrize("paged", [True, False])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
def test_the_same_struct(paged, dtype):
    base = _case(paged, dtype)
    other = [{}, dict(workspace=None), dict(causal=True, scale=1), dict(scale=float("nan")), dict(query_start_loc=None, kv_start_loc=None),
             dict(max_q_len=0, max_kv_len=2 ** 31 - 1), dict(scale=-1e-50), dict(scale=float("inf")), dict(seq_lens=torch.zeros(0, dtype=torch.int32)),
             dict(q=torch.zeros(0, 4, 128, dtype=dtype), out=torch.zeros(0, 4, 128, dtype=dtype)),
             dict(q=torch.zeros(4, 3, 128, dtype=dtype).transpose(0, 1)), dict(q=torch.nn.Parameter(base["q"].clone()))]
    for change in other:
        c = dict(base, **change)
        a = A.AttnArgs(*B._attn_fields(*c.values()))
        assert _pack(c) == bytes(a), change
        assert len(bytes(a)) == ctypes.sizeof(A.AttnArgs)
    x, w, out = torch.zeros(3, 64, dtype=dtype), torch.zeros(64, dtype=dtype), torch.zeros(3, 72, dtype=dtype)[:, :64]
    for res in (None, torch.zeros(3, 64, dtype=dtype)):
        assert F.pack_rmsnorm(x, w, out, 1e-5, res) == bytes(A.make_rmsnorm_args(x, w, out, 1e-5, res))
    kn, cache, slots = torch.zeros(3, 2, 64, dtype=dtype), torch.zeros(4, 16, 2, 64, dtype=dtype), torch.zeros(3, dtype=torch.int32)
    assert F.pack_kv_write(kn, kn, cache, cache, slots) == bytes(A.make_kv_write_args(kn, kn, cache, cache, slots))


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("name,value", [
    ("q", torch.zeros(3, 4, 128, dtype=torch.bfloat16).as_subclass(_Sub)), ("q", torch.zeros(3, 4, 128, dtype=torch.bfloat16).transpose(1, 2)),
    ("q", torch.zeros(12, 128, dtype=torch.bfloat16)), ("out", torch.zeros(3, 4, 128)), ("q", np.zeros((3, 4, 128))),
    ("k", torch.zeros(5, 16, 2, 64, dtype=torch.bfloat16)), ("v", torch.zeros(5, 16, 2, 128, dtype=torch.float16)),
    ("v", torch.zeros(5, 2, 16, 128, dtype=torch.bfloat16).transpose(1, 2)), ("seq_lens", torch.zeros(2, dtype=torch.int64)), ("seq_lens", None),
    ("seq_lens", torch.tensor(3, dtype=torch.int32)), ("block_table", torch.zeros(5, 2, dtype=torch.int32).t()), ("block_table", None),
    ("query_start_loc", torch.zeros(6, dtype=torch.int32)[::2]), ("kv_start_loc", torch.zeros(3)), ("scale", np.float32(0.5)), ("scale", 1e39),
    ("scale", torch.tensor(0.5)), ("scale", True), ("scale", 10 ** 400), ("max_q_len", 3.0), ("max_kv_len", 1 << 31), ("max_kv_len", 1 << 80),
    ("max_kv_len", np.int32(70)), ("max_kv_len", True), ("causal", 1), ("causal", None), ("workspace", 7)])
def test_everything_else_is_left_to_the_general_path(name, value):
    assert _pack(_case()) is not None
    assert _pack(dict(_case(), **{name: value})) is None


def test_modes_wrappers_and_cpu_tensors_are_left_to_the_general_path():
    from torch.overrides import TorchFunctionMode

    class Mode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    c = _case()
    with Mode():
        assert _pack(c) is None
    seen = []

    def f(q):
        seen.append(_pack(dict(_case(), q=q)))  # a batched wrapper: exactly a torch.Tensor, without storage of its own
        return q

    torch.vmap(f)(torch.zeros(2, 3, 4, 128, dtype=torch.bfloat16))
    assert seen == [None]
    assert F.attn(0, *_case().values()) is None  # CPU tensors are never launched with
    kn, cache, slots = torch.zeros(3, 2, 64), torch.zeros(4, 16, 2, 64), torch.zeros(3, dtype=torch.int32)
    assert F.kv_write(kn, kn, cache, cache, slots) is None
    x = torch.zeros(3, 64)
    assert F.rmsnorm(x, x[0], x, 1e-5, None) is None and F.rmsnorm(x, None, x, 1e-5, None) is None
    assert F.pack_rmsnorm(x.t(), x[0], x, 1e-5, None) is None and F.pack_kv_write(kn, torch.zeros(3, 2, 128)[:, :, :64], cache, cache, slots) is None
    with pytest.raises(TypeError):
        F.kv_write(kn)


@pytest.mark.parametrize("name", ["seq_lens", "query_start_loc", "kv_start_loc", "block_table", "workspace", "k", "out"])
def test_a_tensor_elsewhere_than_the_others_is_left_to_the_general_path(name):
    c = _case(paged=name != "kv_start_loc")
    assert _pack(c) is not None
    assert _pack(dict(c, **{name: c[name].to("meta")})) is None


def _host_calls():
    """(what is refused, call) with one small call of every kind, all tensors in host memory."""
    c = _case()
    q = c["q"]
    yield "q", lambda: A.attn_prefill_varlen(q, c["k"], c["v"], c["out"], c["query_start_loc"], c["seq_lens"], 1.0, max_q_len=2, max_kv_len=20,
                                             block_table=c["block_table"])
    yield "q", lambda: A.attn_decode_paged(q, c["k"], c["v"], c["out"], c["block_table"], c["seq_lens"], 1.0, max_kv_len=20)
    yield "q", lambda: A.attn_decode_paged_static(q, c["k"], c["v"], c["out"], c["block_table"], c["seq_lens"], 1.0, max_kv_len=20)
    x = torch.zeros(3, 64, dtype=torch.bfloat16)
    yield "x", lambda: A.rmsnorm_fused_add(x, x[0], x, 1e-5)
    kn, cache, slots = torch.zeros(3, 2, 64), torch.zeros(4, 16, 2, 64), torch.zeros(3, dtype=torch.int32)
    yield "k_new", lambda: A.attn_kv_cache_write(kn, kn, cache, cache, slots)


def test_host_tensors_are_refused_before_a_launch():
    for name, call in _host_calls():
        with pytest.raises(ValueError, match="^%s: " % name):
            call()
    empty = torch.zeros(0, 64, dtype=torch.bfloat16)
    A.rmsnorm_fused_add(empty, torch.zeros(64, dtype=torch.bfloat16), empty, 1e-5, stream=_NoStream)  # nothing to launch


def test_a_bound_is_whatever_int_takes():
    q, kv, i = torch.zeros(0, 4, 128, dtype=torch.bfloat16), torch.zeros(1, 2, 128, dtype=torch.bfloat16), torch.zeros(2, dtype=torch.int32)
    for bound in (8000, 8000.5, "8000", np.int64(8000), torch.tensor(8000), True):
        A.attn_prefill_varlen(q, kv, kv, q, i, i[:1], 1.0, max_q_len=8, max_kv_len=bound, stream=_NoStream)


def test_without_the_extension_the_general_path_takes_every_call():
    """An extension that is missing or built for another torch costs the native path and a warning, not the calls."""
    import os
    import subprocess
    import sys

    here = os.path.dirname(os.path.abspath(__file__))
    code = ("import sys, types; sys.path[:0] = [%r, %r]\n"
            "sys.modules['paper_2505_03780_amd._fastcall'] = None\n"
            "import torch, paper_2505_03780_amd as A\n"
            "from paper_2505_03780_amd import binding as B\n"
            "from test_binding_args import _case, _NoStream\n"
            "c = _case()\n"
            "assert bytes(A.make_args(*[c[n] for n in ('q', 'k', 'v', 'out', 'seq_lens', 'scale')], max_q_len=3, max_kv_len=70, block_table=c['block_table'])) and B._fast is None\n"
            "x = torch.zeros(0, 64, dtype=torch.bfloat16)\n"
            "A.rmsnorm_fused_add(x, torch.zeros(64, dtype=torch.bfloat16), x, 1e-5, stream=_NoStream)\n"
            "q, kv = torch.zeros(0, 4, 128, dtype=torch.bfloat16), torch.zeros(1, 2, 128, dtype=torch.bfloat16)\n"
            "i = torch.zeros(2, dtype=torch.int32)\n"
            "A.attn_prefill_varlen(q, kv, kv, q, i, i[:1], 1.0, max_q_len=8, max_kv_len=8000, stream=_NoStream)\n"
            "print('served')\n" % (os.path.dirname(here), here))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "served" and r.stderr.count("native path cannot be loaded (import") == 1, r.stderr


@pytest.mark.gpu
def test_one_host_tensor_among_device_tensors_is_refused():
    """Nothing is launched with a host pointer: every tensor of a decode and of a prefill call in turn; pinned memory serves."""
    c = {n: t.cuda() if torch.is_tensor(t) else t for n, t in _case().items()}
    c["seq_lens"].fill_(7)
    c["query_start_loc"].copy_(torch.arange(c["query_start_loc"].numel(), dtype=torch.int32))
    c["block_table"].zero_()
    big = torch.zeros(1 << 22, dtype=torch.uint8, device="cuda")
    B_ = c["seq_lens"].shape[0]
    q, out = c["q"][:B_], c["out"][:B_]

    def prefill(d):
        A.attn_prefill_varlen(d["q"], d["k"], d["v"], d["out"], d["query_start_loc"], d["seq_lens"], 1.0, max_q_len=1, max_kv_len=20,
                              block_table=d["block_table"])

    def decode(d):
        A.attn_decode_paged(d["q"], d["k"], d["v"], d["out"], d["block_table"], d["seq_lens"], 1.0, max_kv_len=20, workspace=d["workspace"])

    c.update(q=q, out=out, workspace=big, query_start_loc=torch.arange(B_ + 1, dtype=torch.int32, device="cuda"))
    for call, names in ((prefill, ("q", "k", "v", "out", "query_start_loc", "seq_lens", "block_table")),
                        (decode, ("q", "k", "v", "out", "seq_lens", "block_table", "workspace"))):
        call(c)
        torch.cuda.synchronize()
        want = c["out"].clone()
        for name in names:
            with pytest.raises(ValueError, match="host memory"):
                call(dict(c, **{name: c[name].cpu()}))
        out.zero_()
        torch.cuda.synchronize()
        call(dict(c, seq_lens=c["seq_lens"].cpu().pin_memory()))
        torch.cuda.synchronize()
        assert torch.equal(c["out"], want)


@pytest.mark.gpu
def test_both_paths_give_the_same_result(monkeypatch):
    from attn_testlib import DeviceWorkload
    import workloads as W

    dw = DeviceWorkload(W.make_paged(190, "prefill", [5, 30], [300, 64], 8, 2, 128, 16, 40))
    dec = DeviceWorkload(W.make_paged(191, "decode", [1, 1], [700, 40], 8, 2, 128, 16, 60))
    dec.args(True)
    x, w = torch.randn(5, 1024, device="cuda", dtype=torch.bfloat16), torch.ones(1024, device="cuda", dtype=torch.bfloat16)
    kn, slots = torch.randn(5, 2, 128, device="cuda", dtype=torch.bfloat16), torch.arange(5, dtype=torch.int32, device="cuda") * 3

    def calls():
        for t in (dw.out, dec.out):
            t.fill_(float("nan"))
        y, cache = torch.empty_like(x), torch.zeros(2, 2, 16, 2, 128, device="cuda", dtype=torch.bfloat16)
        A.attn_prefill_varlen(dw.q, dw.k, dw.v, dw.out, dw.qsl, dw.seq_lens, dw.wl.scale, max_q_len=dw.max_q, max_kv_len=dw.max_kv, block_table=dw.bt)
        A.attn_decode_paged(dec.q, dec.k, dec.v, dec.out, dec.bt, dec.seq_lens, dec.wl.scale, max_kv_len=dec.max_kv, workspace=dec.ws)
        first = dec.out.clone()
        A.attn_decode_paged_static(dec.q, dec.k, dec.v, dec.out, dec.bt, dec.seq_lens, dec.wl.scale, max_kv_len=dec.max_kv)
        A.rmsnorm_fused_add(x, w, y, 1e-5)
        A.attn_kv_cache_write(kn, kn, cache[0], cache[1], slots)
        return [dw.out.clone(), first, dec.out.clone(), y, cache]

    native = calls()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # the current stream, whichever it is
        on_side = calls()
    side.synchronize()
    with pytest.raises(A.AttnError):  # the library's refusal comes back as the same error
        A.attn_decode_paged(dec.q, dec.k, dec.v, dec.out, dec.bt, dec.seq_lens, dec.wl.scale, max_kv_len=1 << 20, workspace=dec.ws)
    monkeypatch.setattr(B, "_fast", None)
    for a, b, c in zip(native, on_side, calls()):
        assert torch.equal(a, c) and torch.equal(b, c)
