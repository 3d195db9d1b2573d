"""What the built-in choice of a prefill instance takes without a causal mask, where all tiles of a sequence cost the same (host only)."""
import pytest

import paper_2505_03780_amd as A
from test_prefill_halves import _selected


@pytest.mark.parametrize("d,dtype", [(128, A.ATTN_BF16), (64, A.ATTN_BF16), (128, A.ATTN_F16), (64, A.ATTN_F16)])
def test_order_without_a_causal_mask(d, dtype):
    """Sequences outermost above 2048 keys, and for 32 sequences on."""
    def by_seq(batch, n, causal=0):
        name = _selected(batch, n, n, batch * n, d=d, dtype=dtype, causal=causal, paged=False)
        assert "_ring " in name and "halves" not in name
        return "seqmajor" in name

    assert not by_seq(6, 2048) and by_seq(6, 2049) and by_seq(6, 8192)
    assert not by_seq(31, 1000) and by_seq(32, 1000) and by_seq(32, 400)
    assert not by_seq(4, 2049, causal=1)  # (the small tiles of a triangle stay for the end)
