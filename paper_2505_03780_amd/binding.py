"""Argument marshalling for the C ABI declared in ``include/attn.h`` (same names, no arithmetic).

The operation is the fused attention kernel the paper studies (section "Method and
Investigated Kernels"): causal variable-length prefill and paged-KV decode with grouped-query
heads.  If the shared library has not been built this module raises; there is no fallback.
"""
from __future__ import annotations

import ctypes
import os
import struct
from typing import Optional

ATTN_F32, ATTN_BF16, ATTN_F16 = 0, 1, 2

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libattn_gfx950.so")
_lib = None
_hot = {}  # entry point name -> the same function taking the packed argument struct


class AttnError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__("%s failed: %s (%d)" % (where, attn_status_string(status), status))


class AttnArgs(ctypes.Structure):
    """Mirror of ``struct attn_args``."""

    _fields_ = [
        ("struct_bytes", ctypes.c_uint32),
        ("dtype", ctypes.c_int32),
        ("num_seqs", ctypes.c_int32),
        ("num_q_heads", ctypes.c_int32),
        ("num_kv_heads", ctypes.c_int32),
        ("head_dim", ctypes.c_int32),
        ("total_q", ctypes.c_int32),
        ("max_q_len", ctypes.c_int32),
        ("max_kv_len", ctypes.c_int32),
        ("q", ctypes.c_void_p),
        ("q_stride_tok", ctypes.c_int64),
        ("q_stride_head", ctypes.c_int64),
        ("out", ctypes.c_void_p),
        ("o_stride_tok", ctypes.c_int64),
        ("o_stride_head", ctypes.c_int64),
        ("k", ctypes.c_void_p),
        ("v", ctypes.c_void_p),
        ("kv_stride_block", ctypes.c_int64),
        ("kv_stride_tok", ctypes.c_int64),
        ("kv_stride_head", ctypes.c_int64),
        ("block_table", ctypes.c_void_p),
        ("block_table_stride", ctypes.c_int32),
        ("block_size", ctypes.c_int32),
        ("num_blocks", ctypes.c_int32),
        ("query_start_loc", ctypes.c_void_p),
        ("kv_start_loc", ctypes.c_void_p),
        ("seq_lens", ctypes.c_void_p),
        ("scale", ctypes.c_float),
        ("causal", ctypes.c_int32),
        ("workspace", ctypes.c_void_p),
        ("workspace_bytes", ctypes.c_uint64),
    ]


def library_path() -> str:
    return _LIB_PATH


def load_library():
    """Load the HIP library.  Raises if it has not been built (python -m paper_2505_03780_amd.build)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise ImportError("%s is missing: build it with `python -m paper_2505_03780_amd.build`" % _LIB_PATH)
    lib = ctypes.CDLL(_LIB_PATH)
    P = ctypes.POINTER(AttnArgs)
    lib.attn_prefill_varlen.restype = ctypes.c_int
    lib.attn_prefill_varlen.argtypes = [P, ctypes.c_void_p]
    lib.attn_decode_paged.restype = ctypes.c_int
    lib.attn_decode_paged.argtypes = [P, ctypes.c_void_p]
    lib.attn_decode_paged_static.restype = ctypes.c_int
    lib.attn_decode_paged_static.argtypes = [P, ctypes.c_void_p]
    lib.attn_static_scratch_bytes.restype = ctypes.c_size_t
    lib.attn_static_scratch_bytes.argtypes = []
    lib.attn_workspace_bytes.restype = ctypes.c_size_t
    lib.attn_workspace_bytes.argtypes = [P, ctypes.c_int]
    lib.attn_prefill_scratch_bytes.restype = ctypes.c_size_t
    lib.attn_prefill_scratch_bytes.argtypes = [P]
    lib.attn_prefill_parts_instance.restype = ctypes.c_int
    lib.attn_prefill_parts_instance.argtypes = [P, ctypes.POINTER(ctypes.c_int32)]
    lib.attn_prefill_varlen_parts.restype = ctypes.c_int
    lib.attn_prefill_varlen_parts.argtypes = [P, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    lib.attn_tune.restype = ctypes.c_int
    lib.attn_tune.argtypes = [P, ctypes.c_int, ctypes.c_char_p, ctypes.c_int, ctypes.c_int]
    lib.attn_environment_key.restype = ctypes.c_int
    lib.attn_environment_key.argtypes = [ctypes.c_char_p, ctypes.c_size_t]
    lib.attn_load_cache.restype = ctypes.c_int
    lib.attn_load_cache.argtypes = [ctypes.c_char_p]
    lib.attn_clear_cache.restype = None
    lib.attn_clear_cache.argtypes = []
    lib.attn_num_instances.restype = ctypes.c_int
    lib.attn_num_instances.argtypes = [ctypes.c_int]
    lib.attn_instance_name.restype = ctypes.c_int
    lib.attn_instance_name.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_char_p, ctypes.c_size_t]
    lib.attn_selected_instance.restype = ctypes.c_int
    lib.attn_selected_instance.argtypes = [P, ctypes.c_int]
    lib.attn_force_instance.restype = None
    lib.attn_force_instance.argtypes = [ctypes.c_int, ctypes.c_int]
    lib.attn_status_string.restype = ctypes.c_char_p
    lib.attn_status_string.argtypes = [ctypes.c_int]
    lib.attn_kv_cache_write.restype = ctypes.c_int
    lib.attn_kv_cache_write.argtypes = [ctypes.POINTER(KvWriteArgs), ctypes.c_void_p]
    R = ctypes.POINTER(RmsNormArgs)
    lib.rmsnorm_fused_add.restype = ctypes.c_int
    lib.rmsnorm_fused_add.argtypes = [R, ctypes.c_void_p]
    lib.rmsnorm_tune.restype = ctypes.c_int
    lib.rmsnorm_tune.argtypes = [R, ctypes.c_char_p, ctypes.c_int, ctypes.c_int]
    lib.rmsnorm_num_instances.restype = ctypes.c_int
    lib.rmsnorm_num_instances.argtypes = []
    lib.rmsnorm_instance_name.restype = ctypes.c_int
    lib.rmsnorm_instance_name.argtypes = [ctypes.c_int, ctypes.c_char_p, ctypes.c_size_t]
    lib.rmsnorm_selected_instance.restype = ctypes.c_int
    lib.rmsnorm_selected_instance.argtypes = [R]
    lib.rmsnorm_force_instance.restype = None
    lib.rmsnorm_force_instance.argtypes = [ctypes.c_int]
    # The calls with tensors hand the argument struct over as packed bytes: one struct.pack instead of thirty
    # ctypes field stores (with the checks in one condition and the raw stream handle, a call whose kernel is shorter than its host time takes
    # 5.0-6.6 us instead of 8.3-10.9).
    for name in ("attn_prefill_varlen", "attn_decode_paged", "attn_decode_paged_static", "attn_kv_cache_write", "rmsnorm_fused_add"):
        f = lib[name]  # (a function object of its own: the attribute of that name keeps its argument types)
        f.restype = ctypes.c_int
        f.argtypes = [ctypes.c_char_p, ctypes.c_void_p]
        _hot[name] = f
    f = lib["attn_prefill_scratch_bytes"]
    f.restype = ctypes.c_size_t
    f.argtypes = [ctypes.c_char_p]
    _hot["attn_prefill_scratch_bytes"] = f
    f = lib["attn_prefill_varlen_parts"]
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_char_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p]
    _hot["attn_prefill_varlen_parts"] = f
    _lib = lib
    return lib


class KvWriteArgs(ctypes.Structure):
    """Mirror of ``attn_kv_write_args`` in include/attn.h."""
    _fields_ = [
        ("struct_bytes", ctypes.c_uint32),
        ("dtype", ctypes.c_int32),
        ("num_tokens", ctypes.c_int32),
        ("num_kv_heads", ctypes.c_int32),
        ("head_dim", ctypes.c_int32),
        ("block_size", ctypes.c_int32),
        ("num_blocks", ctypes.c_int32),
        ("reserved", ctypes.c_int32),
        ("k_new", ctypes.c_void_p),
        ("v_new", ctypes.c_void_p),
        ("new_stride_tok", ctypes.c_int64),
        ("new_stride_head", ctypes.c_int64),
        ("k_cache", ctypes.c_void_p),
        ("v_cache", ctypes.c_void_p),
        ("kv_stride_block", ctypes.c_int64),
        ("kv_stride_tok", ctypes.c_int64),
        ("kv_stride_head", ctypes.c_int64),
        ("slot_mapping", ctypes.c_void_p),
    ]


class RmsNormArgs(ctypes.Structure):
    """Mirror of ``rmsnorm_args`` in include/rmsnorm.h."""
    _fields_ = [
        ("struct_bytes", ctypes.c_uint32),
        ("dtype", ctypes.c_int32),
        ("num_tokens", ctypes.c_int32),
        ("hidden", ctypes.c_int32),
        ("x", ctypes.c_void_p),
        ("x_stride", ctypes.c_int64),
        ("residual", ctypes.c_void_p),
        ("residual_stride", ctypes.c_int64),
        ("weight", ctypes.c_void_p),
        ("out", ctypes.c_void_p),
        ("out_stride", ctypes.c_int64),
        ("eps", ctypes.c_float),
    ]


def attn_status_string(status: int) -> str:
    return load_library().attn_status_string(int(status)).decode()


_codes = None
# The native path of the tensor calls (csrc/fast_call.cpp) once torch has been seen: takes plain tensors on the current
# stream, returns the status, or None for a call that the general path below has to decide.  It is tied to one Python and one torch;
# where it cannot be loaded every call goes the general way.
_fast = None


def _dtype_codes():
    """torch dtype -> attn_dtype (torch is imported by the first call that sees a tensor)."""
    global _codes, _int32, _raw_stream, _current_stream, _current_device, _fast
    if _codes is None:
        import torch

        try:
            from . import _fastcall  # (built next to the library, for this Python and torch; needs torch loaded)
        except ImportError as e:
            import warnings

            warnings.warn("the tensor calls' native path cannot be loaded (%s): they are marshalled in Python, and long prefill contexts "
                          "are not split; `python -m paper_2505_03780_amd.build` builds it for this torch" % e)
        else:
            lib = load_library()
            address = lambda name: ctypes.cast(getattr(lib, name), ctypes.c_void_p).value
            _fastcall.bind(*(address(name) for name in ("attn_prefill_varlen", "attn_decode_paged", "attn_decode_paged_static",
                                                        "attn_kv_cache_write", "rmsnorm_fused_add")))
            _fast = _fastcall

        _int32 = torch.int32
        _current_stream, _current_device = torch.cuda.current_stream, torch.cuda.current_device
        _raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)  # (current_stream() builds a Python object)
        _codes = {torch.bfloat16: ATTN_BF16, torch.float32: ATTN_F32, torch.float16: ATTN_F16}
    return _codes


def _dtype_code(t) -> int:
    code = _dtype_codes().get(t.dtype)
    if code is None:
        raise TypeError("tensors must be bfloat16, float16 or float32")
    return code


def _refuse_attn(q, k, v, out, seq_lens, query_start_loc, kv_start_loc, block_table):
    """Raises for the first check of an attention call that fails."""
    for name, t in (("q", q), ("k", k), ("v", v), ("out", out)):
        if t.stride(-1) != 1:
            raise ValueError("%s: head_dim must be contiguous" % name)
    for name, t in (("seq_lens", seq_lens), ("query_start_loc", query_start_loc), ("kv_start_loc", kv_start_loc),
                    ("block_table", block_table)):
        if t is not None and (t.dtype != _int32 or not t.is_contiguous()):
            raise TypeError("%s must be a contiguous int32 tensor" % name)
    if k.dtype != q.dtype or v.dtype != q.dtype or out.dtype != q.dtype:
        raise TypeError("q, k, v, out must share a dtype")
    if k.stride() != v.stride() or k.shape != v.shape:
        raise ValueError("k and v must have the same shape and strides")
    _dtype_code(q)


def _attn_fields(q, k, v, out, seq_lens, scale, max_q_len, max_kv_len, query_start_loc, kv_start_loc, block_table, causal, workspace):
    """The checked field values of an AttnArgs, in order (null pointers as 0)."""
    codes = _codes or _dtype_codes()
    qs, ks, os_ = q.stride(), k.stride(), out.stride()
    dtype, qshape, kshape = q.dtype, q.shape, k.shape
    code = codes.get(dtype)
    # (one condition over all checks: the loops that name the culprit only run for a call that is wrong)
    if (qs[-1] != 1 or ks[-1] != 1 or os_[-1] != 1 or v.stride() != ks or v.shape != kshape or code is None
            or k.dtype != dtype or v.dtype != dtype or out.dtype != dtype
            or seq_lens.dtype != _int32 or not seq_lens.is_contiguous()
            or (query_start_loc is not None and (query_start_loc.dtype != _int32 or not query_start_loc.is_contiguous()))
            or (kv_start_loc is not None and (kv_start_loc.dtype != _int32 or not kv_start_loc.is_contiguous()))
            or (block_table is not None and (block_table.dtype != _int32 or not block_table.is_contiguous()))):
        _refuse_attn(q, k, v, out, seq_lens, query_start_loc, kv_start_loc, block_table)
    if block_table is not None:
        if len(kshape) != 4:
            raise ValueError("paged k/v must be [num_blocks, block_size, Hkv, D]")
        num_blocks, block_size, hkv, _ = kshape
        kv_block, kv_tok, kv_head, _ = ks
        table, table_stride = block_table.data_ptr(), block_table.stride(0)
    else:
        if len(kshape) != 3:
            raise ValueError("contiguous k/v must be [total_kv, Hkv, D]")
        hkv = kshape[1]
        kv_block, kv_tok, kv_head = 0, ks[0], ks[1]
        table = table_stride = block_size = num_blocks = 0
    if workspace is None:
        ws = ws_bytes = 0
    else:
        ws, ws_bytes = workspace.data_ptr(), workspace.nbytes
    return (_ATTN_BYTES, code, seq_lens.shape[0], qshape[1], hkv, qshape[2], qshape[0], int(max_q_len), int(max_kv_len),
            q.data_ptr(), qs[0], qs[1], out.data_ptr(), os_[0], os_[1], k.data_ptr(), v.data_ptr(), kv_block, kv_tok, kv_head,
            table, table_stride, block_size, num_blocks,
            0 if query_start_loc is None else query_start_loc.data_ptr(), 0 if kv_start_loc is None else kv_start_loc.data_ptr(),
            seq_lens.data_ptr(), float(scale), 1 if causal else 0, ws, ws_bytes)


_ATTN_BYTES = ctypes.sizeof(AttnArgs)
_pack_attn = struct.Struct("@I8iPqqPqqPPqqqPiiiPPPfiPQ").pack
_pack_kv_write = struct.Struct("@I7iPPqqPPqqqP").pack
_pack_rmsnorm = struct.Struct("@IiiiPqPqPPqf4x").pack


def _packed(pack, cls, fields) -> bytes:
    try:
        return pack(*fields)
    except (struct.error, OverflowError):  # a value that does not fit its field: ctypes' conversion decides
        return bytes(cls(*fields))


def make_args(q, k, v, out, seq_lens, scale, *, max_q_len, max_kv_len, query_start_loc=None, kv_start_loc=None,
              block_table=None, causal=True, workspace=None, is_decode=False) -> AttnArgs:
    """Fill an AttnArgs from device tensors.  q/out: [total_q, Hq, D]; k/v: [total_kv, Hkv, D] or,
    with block_table, [num_blocks, block_size, Hkv, D].  Only strides and pointers are read."""
    return AttnArgs(*_attn_fields(q, k, v, out, seq_lens, scale, max_q_len, max_kv_len, query_start_loc, kv_start_loc, block_table,
                                  causal, workspace))


def _stream_ptr(stream) -> int:
    if stream is not None:
        return int(stream.cuda_stream)
    if _codes is None:
        _dtype_codes()
    if _raw_stream is None:
        return int(_current_stream().cuda_stream)
    return _raw_stream(_current_device())


def _refuse_host_tensors(names, *tensors):
    """Raises for a tensor in host memory that kernels cannot read (a launch with it would fault the GPU); pinned memory they can."""
    if _fast is not None and not _fast.any_on_host(*tensors):
        return
    named = dict(zip(names.split(), tensors))
    if any(len(t) == 0 for t in (tensors[0], named.get("seq_lens")) if t is not None):
        return  # nothing to launch
    for name, t in named.items():
        if t is not None and getattr(t, "is_cpu", False) and t.numel() > 0 and not t.is_pinned():
            raise ValueError("%s: a tensor on the GPU is needed, this one is in host memory" % name)


def _prefill_scratch(packed: bytes, stream):
    """(address, bytes) of scratch memory for the prefill call described by ``packed`` on ``stream``; (0, 0) for a call that does
    without: one that uses none, on a stream that is not torch's or not the current device's, under capture, when memory is short, or
    without the native path, which takes the memory."""
    n = _hot["attn_prefill_scratch_bytes"](packed) if _fast is not None else 0
    if n == 0:
        return 0, 0
    if stream is not None:
        import torch

        if not isinstance(stream, torch.cuda.Stream) or stream.device_index != _current_device():
            return 0, 0
    return _fast.scratch(n, _stream_ptr(stream)), n


def attn_prefill_varlen(q, k, v, out, query_start_loc, seq_lens, scale, *, max_q_len, max_kv_len, causal=True,
                        block_table=None, kv_start_loc=None, stream=None, args: Optional[AttnArgs] = None, workspace=None) -> None:
    """Enqueue causal variable-length (or chunked, over a paged prefix) prefill on ``stream``.

    The keys of few query rows over many keys are split over the whole GPU, which takes scratch memory.  ``workspace`` is a
    16-byte aligned device tensor for that, of at least attn_prefill_scratch_bytes; a smaller one is not used.  Without it a call
    with tensors takes memory from torch's caching allocator for its time on the stream, but for a call under graph capture, where
    nobody would hold the memory for the replays, and a call with ``args`` does without.  The result is the same within rounding."""
    lib = _lib or load_library()
    rc = None
    if args:
        if workspace is None:
            rc = lib.attn_prefill_varlen(ctypes.byref(args), _stream_ptr(stream))
        else:
            _refuse_host_tensors("workspace", workspace)
            rc = lib.attn_prefill_varlen_parts(ctypes.byref(args), workspace.data_ptr(), workspace.nbytes, _stream_ptr(stream))
    elif _fast is not None and stream is None and int(max_kv_len) <= 1024:  # (longer ones may use scratch memory)
        rc = _fast.attn(0, q, k, v, out, seq_lens, scale, max_q_len, max_kv_len, query_start_loc, kv_start_loc, block_table, causal, None)
    if rc is None:
        a = _packed(_pack_attn, AttnArgs, _attn_fields(q, k, v, out, seq_lens, scale, max_q_len, max_kv_len, query_start_loc, kv_start_loc,
                                                       block_table, causal, None))
        _refuse_host_tensors("q k v out query_start_loc seq_lens block_table kv_start_loc workspace", q, k, v, out, query_start_loc, seq_lens,
                             block_table, kv_start_loc, workspace)
        ptr = 0
        if workspace is not None:
            rc = _hot["attn_prefill_varlen_parts"](a, workspace.data_ptr(), workspace.nbytes, _stream_ptr(stream))
        # (necessary conditions of the library's own rule, to save short calls the question)
        elif int(max_kv_len) > 1024 and q.shape[0] * q.shape[1] <= 131072:
            ptr, n = _prefill_scratch(a, stream)
        if ptr:
            try:
                rc = _hot["attn_prefill_varlen_parts"](a, ptr, n, _stream_ptr(stream))
            finally:
                _fast.release(ptr)
        elif rc is None:
            rc = _hot["attn_prefill_varlen"](a, _stream_ptr(stream))
    if rc != 0:
        raise AttnError(rc, "attn_prefill_varlen")


def attn_decode_paged(q, k_cache, v_cache, out, block_table, seq_lens, scale, *, max_kv_len, workspace=None, stream=None,
                      args: Optional[AttnArgs] = None) -> None:
    """Enqueue paged-KV decode (one query token per sequence) on ``stream``."""
    lib = _lib or load_library()
    rc = None
    if args:
        rc = lib.attn_decode_paged(ctypes.byref(args), _stream_ptr(stream))
    elif _fast is not None and stream is None:
        rc = _fast.attn(1, q, k_cache, v_cache, out, seq_lens, scale, 1, max_kv_len, None, None, block_table, True, workspace)
    if rc is None:
        a = _packed(_pack_attn, AttnArgs, _attn_fields(q, k_cache, v_cache, out, seq_lens, scale, 1, max_kv_len, None, None, block_table,
                                                       True, workspace))
        _refuse_host_tensors("q k_cache v_cache out block_table seq_lens workspace", q, k_cache, v_cache, out, block_table, seq_lens, workspace)
        rc = _hot["attn_decode_paged"](a, _stream_ptr(stream))
    if rc != 0:
        raise AttnError(rc, "attn_decode_paged")


def attn_decode_paged_static(q, k_cache, v_cache, out, block_table, seq_lens, scale, *, max_kv_len, stream=None,
                             args: Optional[AttnArgs] = None) -> None:
    """attn_decode_paged with the split-K records in the library's own static device array: no workspace
    argument, nothing allocated."""
    lib = _lib or load_library()
    rc = None
    if args:
        rc = lib.attn_decode_paged_static(ctypes.byref(args), _stream_ptr(stream))
    elif _fast is not None and stream is None:
        rc = _fast.attn(2, q, k_cache, v_cache, out, seq_lens, scale, 1, max_kv_len, None, None, block_table, True, None)
    if rc is None:
        a = _packed(_pack_attn, AttnArgs, _attn_fields(q, k_cache, v_cache, out, seq_lens, scale, 1, max_kv_len, None, None, block_table,
                                                       True, None))
        _refuse_host_tensors("q k_cache v_cache out block_table seq_lens", q, k_cache, v_cache, out, block_table, seq_lens)
        rc = _hot["attn_decode_paged_static"](a, _stream_ptr(stream))
    if rc != 0:
        raise AttnError(rc, "attn_decode_paged_static")


def attn_static_scratch_bytes() -> int:
    return int(load_library().attn_static_scratch_bytes())


def attn_workspace_bytes(args: AttnArgs, is_decode: bool) -> int:
    return int(load_library().attn_workspace_bytes(ctypes.byref(args), 1 if is_decode else 0))


def attn_prefill_scratch_bytes(args: AttnArgs) -> int:
    return int(load_library().attn_prefill_scratch_bytes(ctypes.byref(args)))


def attn_prefill_parts_instance(args: AttnArgs):
    """(instance, parts of the keys) that the next prefill call with these args and scratch memory would launch."""
    parts = ctypes.c_int32(1)
    rc = int(load_library().attn_prefill_parts_instance(ctypes.byref(args), ctypes.byref(parts)))
    if rc < 0:
        raise AttnError(rc, "attn_prefill_parts_instance")
    return rc, parts.value


def attn_tune(args: AttnArgs, is_decode: bool, cache_path: Optional[str] = None, iters: int = 20, flags: int = 0) -> None:
    path = None if cache_path is None else os.fsencode(cache_path)
    rc = load_library().attn_tune(ctypes.byref(args), 1 if is_decode else 0, path, int(iters), int(flags))
    if rc != 0:
        raise AttnError(rc, "attn_tune")


def attn_environment_key() -> str:
    buf = ctypes.create_string_buffer(256)
    load_library().attn_environment_key(buf, len(buf))
    return buf.value.decode()


def attn_load_cache(cache_path: str) -> int:
    return int(load_library().attn_load_cache(os.fsencode(cache_path)))


def attn_clear_cache() -> None:
    load_library().attn_clear_cache()


def attn_num_instances(is_decode: bool) -> int:
    return int(load_library().attn_num_instances(1 if is_decode else 0))


def attn_instance_name(is_decode: bool, idx: int) -> str:
    buf = ctypes.create_string_buffer(128)
    rc = load_library().attn_instance_name(1 if is_decode else 0, int(idx), buf, 128)
    if rc < 0:
        raise AttnError(rc, "attn_instance_name")
    return buf.value.decode()


def attn_selected_instance(args: AttnArgs, is_decode: bool) -> int:
    return int(load_library().attn_selected_instance(ctypes.byref(args), 1 if is_decode else 0))


def attn_force_instance(is_decode: bool, idx: int) -> None:
    load_library().attn_force_instance(1 if is_decode else 0, int(idx))


# ---- fused RMS layer norm (include/rmsnorm.h) ------------------------------------------------------

def _rmsnorm_fields(x, weight, out, eps, residual):
    """The checked field values of an RmsNormArgs, in order."""
    codes = _codes or _dtype_codes()
    xs, os_ = x.stride(), out.stride()
    rs = None if residual is None else residual.stride()
    for name, st in (("x", xs), ("out", os_), ("residual", rs), ("weight", None if weight is None else weight.stride())):
        if st is not None and st[-1] != 1:
            raise ValueError("%s: the hidden dimension must be contiguous" % name)
    code = codes.get(x.dtype)
    if code is None:
        raise TypeError("tensors must be bfloat16, float16 or float32")
    tokens, hidden = x.shape[:2]
    return (_RMSNORM_BYTES, code, tokens, hidden, x.data_ptr(), xs[0], 0 if residual is None else residual.data_ptr(),
            0 if rs is None else rs[0], 0 if weight is None else weight.data_ptr(), out.data_ptr(), os_[0], float(eps))


_RMSNORM_BYTES = ctypes.sizeof(RmsNormArgs)


def make_rmsnorm_args(x, weight, out, eps, residual=None) -> RmsNormArgs:
    """x, out, residual: [T, H] device tensors with a contiguous last dimension; weight: [H]."""
    return RmsNormArgs(*_rmsnorm_fields(x, weight, out, eps, residual))


def rmsnorm_fused_add(x, weight, out, eps, residual=None, stream=None, args: Optional[RmsNormArgs] = None) -> None:
    """Enqueue out = rmsnorm(x + residual) * weight and residual <- x + residual (residual optional)."""
    lib = _lib or load_library()
    rc = None
    if args:
        rc = lib.rmsnorm_fused_add(ctypes.byref(args), _stream_ptr(stream))
    elif _fast is not None and stream is None:
        rc = _fast.rmsnorm(x, weight, out, eps, residual)
    if rc is None:
        a = _packed(_pack_rmsnorm, RmsNormArgs, _rmsnorm_fields(x, weight, out, eps, residual))
        if weight is not None:  # (a missing weight is the library's to refuse)
            _refuse_host_tensors("x weight out residual", x, weight, out, residual)
        rc = _hot["rmsnorm_fused_add"](a, _stream_ptr(stream))
    if rc != 0:
        raise AttnError(rc, "rmsnorm_fused_add")


def rmsnorm_tune(args: RmsNormArgs, cache_path: Optional[str] = None, iters: int = 20, flags: int = 0) -> None:
    path = None if cache_path is None else os.fsencode(cache_path)
    rc = load_library().rmsnorm_tune(ctypes.byref(args), path, int(iters), int(flags))
    if rc != 0:
        raise AttnError(rc, "rmsnorm_tune")


def rmsnorm_num_instances() -> int:
    return int(load_library().rmsnorm_num_instances())


def rmsnorm_instance_name(idx: int) -> str:
    buf = ctypes.create_string_buffer(128)
    n = load_library().rmsnorm_instance_name(int(idx), buf, len(buf))
    if n < 0:
        raise AttnError(n, "rmsnorm_instance_name")
    return buf.value.decode()


def rmsnorm_selected_instance(args: RmsNormArgs) -> int:
    return int(load_library().rmsnorm_selected_instance(ctypes.byref(args)))


def rmsnorm_force_instance(idx: int) -> None:
    load_library().rmsnorm_force_instance(int(idx))


# ---- KV-cache write ----------------------------------------------------------------------------------

def _kv_write_fields(k_new, v_new, k_cache, v_cache, slot_mapping):
    """The checked field values of a KvWriteArgs, in order."""
    codes = _codes or _dtype_codes()
    if slot_mapping.dtype != _int32 or not slot_mapping.is_contiguous():
        raise TypeError("slot_mapping must be a contiguous int32 tensor")
    kn, vn, kc, vc = k_new.stride(), v_new.stride(), k_cache.stride(), v_cache.stride()
    for name, st in (("k_new", kn), ("v_new", vn), ("k_cache", kc), ("v_cache", vc)):
        if st[-1] != 1:
            raise ValueError("%s: head_dim must be contiguous" % name)
    if kn != vn or kc != vc:
        raise ValueError("K and V must share their strides")
    code = codes.get(k_new.dtype)
    if code is None:
        raise TypeError("tensors must be bfloat16, float16 or float32")
    tokens, hkv, d = k_new.shape[:3]
    num_blocks, block_size = k_cache.shape[:2]
    return (_KV_WRITE_BYTES, code, tokens, hkv, d, block_size, num_blocks, 0, k_new.data_ptr(), v_new.data_ptr(), kn[0], kn[1],
            k_cache.data_ptr(), v_cache.data_ptr(), kc[0], kc[1], kc[2], slot_mapping.data_ptr())


_KV_WRITE_BYTES = ctypes.sizeof(KvWriteArgs)


def make_kv_write_args(k_new, v_new, k_cache, v_cache, slot_mapping) -> KvWriteArgs:
    """k_new, v_new: [T, Hkv, D]; caches: [num_blocks, block_size, Hkv, D]; slot_mapping: int32 [T]."""
    return KvWriteArgs(*_kv_write_fields(k_new, v_new, k_cache, v_cache, slot_mapping))


def attn_kv_cache_write(k_new, v_new, k_cache, v_cache, slot_mapping, stream=None, args: Optional[KvWriteArgs] = None) -> None:
    """Enqueue the scatter of new keys/values into the paged caches."""
    lib = _lib or load_library()
    rc = None
    if args:
        rc = lib.attn_kv_cache_write(ctypes.byref(args), _stream_ptr(stream))
    elif _fast is not None and stream is None:
        rc = _fast.kv_write(k_new, v_new, k_cache, v_cache, slot_mapping)
    if rc is None:
        a = _packed(_pack_kv_write, KvWriteArgs, _kv_write_fields(k_new, v_new, k_cache, v_cache, slot_mapping))
        _refuse_host_tensors("k_new v_new k_cache v_cache slot_mapping", k_new, v_new, k_cache, v_cache, slot_mapping)
        rc = _hot["attn_kv_cache_write"](a, _stream_ptr(stream))
    if rc != 0:
        raise AttnError(rc, "attn_kv_cache_write")
