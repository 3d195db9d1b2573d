"""Host test: which kernels the built-in choice gives to caches with rows or blocks so far apart that 32-bit offsets do not reach."""
import pytest

import paper_2505_03780_amd as A
from test_host_api import _args, _paged


def _name(a, is_decode=False):
    i = A.attn_selected_instance(a, is_decode)
    return A.attn_instance_name(is_decode, i) if i >= 0 else ""


@pytest.mark.parametrize("D", [64, 128])
def test_the_choice_follows_the_strides_from_call_to_call(D):
    """The choice of one call is not handed to the next that differs in its strides alone."""
    A.attn_clear_cache()
    A.attn_force_instance(False, -1)
    for kw in (dict(max_q_len=100, max_kv_len=100), dict(num_seqs=2, max_q_len=16, max_kv_len=8000)):  # ring, key split
        near, far = _args(head_dim=D, **kw), _args(head_dim=D, kv_stride_tok=1 << 27, **kw)
        first = _name(near)
        assert "ring" in first or "keysplit" in first
        staged = _name(far)
        assert staged and "ring" not in staged and "keysplit" not in staged
        assert _name(near) == first
    near, far = (_paged(head_dim=D, max_q_len=600, max_kv_len=900, kv_stride_block=x) for x in (1 << 20, 1 << 31))
    assert "ring" in _name(near) and "ring" not in _name(far) and "ring" in _name(near)


@pytest.mark.parametrize("dtype", [A.ATTN_BF16, A.ATTN_F16])
@pytest.mark.parametrize("D", [64, 128])
def test_decode_kernels_with_32_bit_row_offsets_are_not_taken_for_rows_far_apart(D, dtype):
    A.attn_clear_cache()
    A.attn_force_instance(True, -1)
    kw = dict(head_dim=D, dtype=dtype, block_table_stride=4096, num_blocks=1 << 20, max_q_len=1)
    for B, kv in ((16, 8000), (128, 400), (64, 30000), (1, 100), (600, 3000)):
        a = _paged(num_seqs=B, total_q=B, max_kv_len=kv, kv_stride_tok=1 << 27, kv_stride_block=1 << 31, **kw)  # 256 MiB between rows
        name = _name(a, True)
        assert name and "balanced" not in name and "_seq" not in name
        near = _paged(num_seqs=B, total_q=B, max_kv_len=kv, kv_stride_tok=(1 << 27) - 8, kv_stride_block=1 << 31, **kw)
        assert _name(near, True) == _name(_paged(num_seqs=B, total_q=B, max_kv_len=kv, **kw), True)
        for i in range(A.attn_num_instances(True)):
            name = A.attn_instance_name(True, i)
            if "balanced" in name or "_seq" in name:
                A.attn_force_instance(True, i)
                assert A.attn_selected_instance(a, True) < 0
        A.attn_force_instance(True, -1)
