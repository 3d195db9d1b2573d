"""Host test of the built-in decode choice at the lines of its rule, for both element types and head sizes."""
import pytest

import paper_2505_03780_amd as A
from test_host_api import _paged


def _name(B, kv, Hq=32, Hkv=8, D=128, dtype=A.ATTN_BF16):
    A.attn_clear_cache()
    A.attn_force_instance(True, -1)
    a = _paged(num_seqs=B, total_q=B, max_q_len=1, max_kv_len=kv, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, dtype=dtype,
               block_table_stride=4096, num_blocks=1 << 20)
    return A.attn_instance_name(True, A.attn_selected_instance(a, True)).replace("decode_bf16", "").replace("decode_f16", "").strip()


@pytest.mark.parametrize("dtype", [A.ATTN_BF16, A.ATTN_F16])
@pytest.mark.parametrize("D,unsplit", [(128, 640), (64, 896)])
def test_lines_of_the_rule(dtype, D, unsplit):
    n = lambda *a, **k: _name(*a, D=D, dtype=dtype, **k)
    d = "d%d " % D
    # short contexts are not split, in workgroups of four wavefronts up to 128 keys
    assert n(1, 128) == d + "w4 split0" and n(1, 129) == d + "w8 split0"
    assert n(1, unsplit) == d + "w8 split0" and n(1, unsplit + 1) == d + "w8 split256"
    assert n(4, 2048) == d + "w8 split256" and n(4, 2049) == d + "w4 split256"  # a compute unit for every part
    assert n(1, 4095) == d + "w8 split256" and n(1, 4096) == d + "w4 split256"
    assert n(16, 1024) == d + "w8 split0" and n(16, 1025) == d + "w4 split256"
    assert n(32, 512) == d + "w4 split0"  # a unit for every compute unit
    # many short contexts: one wavefront per head
    assert n(128, 512) == "_seq " + d + "w4 split512" and n(127, 512) == d + "w4 split0"
    assert n(64, 64) == "_seq " + d + "w4 split512" and n(64, 65) == d + "w4 split0"
    # long runs: from 500 000 keys over the heads on, above 8192 keys from 100 000 keys of the batch on
    assert "balanced" in n(16, 3907) and "split256" in n(16, 3906)
    assert "balanced" in n(11, 9091) and "split" in n(10, 9091)
    # one or two KV heads: never balanced, but for contexts too many to split
    assert "split" in n(40, 4000, Hq=8, Hkv=2) and "balanced" in n(200, 20000, Hq=8, Hkv=2)


def test_balanced_records_stay_within_the_static_array_where_splits_ran_before():
    """50 contexts of 1300 keys: under 128 query heads the balanced kernel's records exceed the 16 MiB array."""
    assert _name(50, 1300, Hq=128) == "d128 w4 split256" and "balanced" in _name(50, 1300, Hq=64)


def test_long_parts_of_few_heads():
    """fp16, D = 64: where the batch's bound leaves parts of 1024 keys or more, the token-balanced kernel (whole-context skew)."""
    n = lambda B, kv, **k: _name(B, kv, D=64, dtype=A.ATTN_F16, **k)
    two = dict(Hq=8, Hkv=2)
    assert "balanced" in n(175, 3338, **two) and "balanced" in n(120, 9000, **two) and "balanced" in n(200, 1800, **two)
    assert "split512" in n(130, 1300, **two)  # parts shorter than 1024 keys
    assert "split" in n(175, 3338, Hq=4, Hkv=1)
    assert _name(175, 3338, D=128, dtype=A.ATTN_F16, **two) == "d128 w4 split2048"
