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
