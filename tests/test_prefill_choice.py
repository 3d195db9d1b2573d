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


@pytest.mark.parametrize("dtype", [A.ATTN_BF16, A.ATTN_F16])
def test_workgroup_without_a_causal_mask(dtype):
    """D = 128 between 2048 and 8192 keys: the small workgroup where it saves half a round (8 tiles for every 32 tokens, 512 places for
    small ones and 256 for large ones), or a tenth of the rows."""
    def small(batch, max_q, max_kv, total, causal=0):
        name = _selected(batch, max_q, max_kv, total, dtype=dtype, causal=causal)
        assert "_ring " in name and "halves" not in name
        return " w4 " in name

    one = lambda n: small(1, n, n, n)
    assert one(2048) and one(3072) and not one(3073) and not one(4096) and one(4097) and one(5120) and not one(5121)
    assert small(2, 4096, 8191, 5000) and not small(2, 4096, 8192, 5000)  # (5.0 against three rounds)
    # 20 tokens to a tile of 32, or to one of 64: a half of the large tiles is padding
    assert small(64, 20, 4096, 64 * 20) and not small(32, 64, 4096, 32 * 64)
    # the same maxima and nearly the same tiles, one round of the large ones or more: other calls, in turn
    for _ in range(2):
        assert not small(3, 1000, 3000, 1919) and small(3, 1000, 3000, 1920)
