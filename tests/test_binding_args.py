"""The packed argument structs of the tensor calls are those that ctypes builds field by field, and a wrong call is refused
with the error of the first check that fails.  No GPU: the structs hold CPU pointers and nothing is called with them."""
import ctypes

import pytest
import torch

import paper_2505_03780_amd as A
from paper_2505_03780_amd import binding as B


class _NoStream:
    cuda_stream = 0


def _case(paged=True, dtype=torch.bfloat16):
    q = torch.zeros(3, 4, 136, dtype=dtype)[:, :, :128]
    kv = (torch.zeros(5, 16, 2, 128, dtype=dtype), torch.zeros(5, 16, 2, 128, dtype=dtype)) if paged else \
        (torch.zeros(7, 2, 128, dtype=dtype), torch.zeros(7, 2, 128, dtype=dtype))
    i32 = lambda *n: torch.zeros(*n, dtype=torch.int32)
    return dict(q=q, k=kv[0], v=kv[1], out=torch.zeros(3, 4, 128, dtype=dtype), seq_lens=i32(2), scale=0.125, max_q_len=3, max_kv_len=70,
                query_start_loc=i32(3), kv_start_loc=None if paged else i32(3), block_table=i32(2, 5) if paged else None, causal=False,
                workspace=torch.zeros(100, dtype=torch.float32))


@pytest.mark.parametrize("paged", [True, False])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
def test_packed_struct_is_the_ctypes_struct(paged, dtype):
    A.load_library()
    c = _case(paged, dtype)
    a = A.make_args(c["q"], c["k"], c["v"], c["out"], c["seq_lens"], c["scale"], **{n: x for n, x in c.items() if n not in ("q", "k", "v", "out", "seq_lens", "scale")})
    fields = B._attn_fields(*c.values())
    assert B._pack_attn(*fields) == bytes(a) and len(bytes(a)) == ctypes.sizeof(A.AttnArgs)
    assert (a.num_seqs, a.num_q_heads, a.num_kv_heads, a.head_dim, a.total_q, a.max_q_len, a.max_kv_len) == (2, 4, 2, 128, 3, 3, 70)
    assert (a.q, a.q_stride_tok, a.q_stride_head, a.o_stride_tok) == (c["q"].data_ptr(), 544, 136, 512)
    assert (a.kv_stride_block, a.kv_stride_tok, a.kv_stride_head) == ((4096, 256, 128) if paged else (0, 256, 128))
    assert (a.block_table_stride, a.block_size, a.num_blocks) == ((5, 16, 5) if paged else (0, 0, 0))
    assert a.causal == 0 and a.workspace_bytes == 400 and a.scale == 0.125
    # a value beyond its field goes through ctypes' conversion, as it did
    wide = list(fields)
    wide[8] = (1 << 32) + 9
    assert A.AttnArgs.from_buffer_copy(B._packed(B._pack_attn, A.AttnArgs, wide)).max_kv_len == 9

    x, w, out = torch.zeros(3, 64, dtype=dtype), torch.zeros(64, dtype=dtype), torch.zeros(3, 72, dtype=dtype)[:, :64]
    for res in (None, torch.zeros(3, 64, dtype=dtype)):
        assert B._pack_rmsnorm(*B._rmsnorm_fields(x, w, out, 1e-5, res)) == bytes(A.make_rmsnorm_args(x, w, out, 1e-5, res))
    kn, cache, slots = torch.zeros(3, 2, 64, dtype=dtype), torch.zeros(4, 16, 2, 64, dtype=dtype), torch.zeros(3, dtype=torch.int32)
    assert B._pack_kv_write(*B._kv_write_fields(kn, kn, cache, cache, slots)) == bytes(A.make_kv_write_args(kn, kn, cache, cache, slots))


@pytest.mark.parametrize("name,value,error", [
    ("q", torch.zeros(3, 4, 128, dtype=torch.bfloat16).transpose(1, 2), ValueError), ("out", torch.zeros(3, 4, 128), TypeError),
    ("k", torch.zeros(5, 16, 2, 64, dtype=torch.bfloat16), ValueError), ("v", torch.zeros(5, 16, 2, 128, dtype=torch.float16), TypeError),
    ("seq_lens", torch.zeros(2, dtype=torch.int64), TypeError), ("block_table", torch.zeros(5, 2, dtype=torch.int32).t(), TypeError),
    ("query_start_loc", torch.zeros(6, dtype=torch.int32)[::2], TypeError), ("kv_start_loc", torch.zeros(3), TypeError)])
def test_wrong_arguments_are_refused(name, value, error):
    c = dict(_case(), **{name: value})
    with pytest.raises(error):
        B._attn_fields(*c.values())
    with pytest.raises(A.AttnError):  # a missing weight is the library's to refuse
        A.rmsnorm_fused_add(torch.zeros(1, 64, dtype=torch.bfloat16), None, torch.zeros(1, 64, dtype=torch.bfloat16), 1e-5, stream=_NoStream)
    for bad in (torch.float64, torch.int16):
        with pytest.raises(TypeError):
            B._attn_fields(*_case(dtype=bad).values())
