"""The ring kernel with two wavefront groups per tile ("halves"): where the built-in choice takes it (host only), and what infinities
among the values do to it, against the workgroup that walks all keys of a tile.  (Its results over every loop and edge are
covered with the other ring instances in test_gpu_ring_starts.py, test_gpu_ring_d128.py and test_gpu_ring_d64.py.)"""
import ctypes
import math
import os
import subprocess
import sys

import pytest
import torch

import paper_2505_03780_amd as A


def _selected(batch, max_q, max_kv, total_q, hq=32, hkv=8, d=128, dtype=A.ATTN_BF16, causal=1, paged=True):
    a = A.AttnArgs()
    a.struct_bytes = ctypes.sizeof(A.AttnArgs)
    a.dtype, a.num_seqs, a.num_q_heads, a.num_kv_heads, a.head_dim = dtype, batch, hq, hkv, d
    a.total_q, a.max_q_len, a.max_kv_len, a.causal = total_q, max_q, max_kv, causal
    a.kv_stride_tok, a.kv_stride_head = hkv * d, d
    if paged:
        a.block_table, a.block_table_stride, a.block_size, a.kv_stride_block = 0x3000, 1 << 12, 16, 16 * hkv * d
    return A.attn_instance_name(False, A.attn_selected_instance(a, False))


@pytest.mark.parametrize("d,dtype", [(128, A.ATTN_BF16), (64, A.ATTN_BF16), (128, A.ATTN_F16), (64, A.ATTN_F16)])
def test_where_halves_are_chosen(d, dtype):
    pick = lambda *a, **k: _selected(*a, d=d, dtype=dtype, **k)
    for hq, hkv, hpw, tok in ((32, 8, 4, 32), (16, 8, 2, 64), (8, 8, 1, 128)):  # 8 workgroups a tile of `tok` tokens
        h = dict(hq=hq, hkv=hkv)
        name = "hpw%d slots4 pf4 halves seqmajor" % hpw
        # 4 sequences: 28 tiles and one more each for uneven lengths, 256 workgroups; one token tile more does not fit
        assert name in pick(4, 10 * tok, 1400, 28 * tok, **h)
        assert "halves" not in pick(4, 10 * tok, 1400, 29 * tok, **h)
        assert name in pick(4, 10 * tok, 8191, 28 * tok, **h) and "halves" not in pick(4, 10 * tok, 8192, 28 * tok, **h)
        # one whole prompt: up to two tiles per compute unit; behind a prefix, or two of them: one
        n = 64 * tok
        assert name in pick(1, n, n, n, **h) and "halves" not in pick(1, n + 1, n + 1, n + 1, **h)
        assert "halves" not in pick(1, n, n + 1, n, **h) and "halves" not in pick(2, n // 2, n // 2, n, **h)
        assert "halves" not in pick(1, n, n, n, causal=0, **h)
    assert "halves" in pick(6, 300, 700, 700) and "halves" not in pick(6, 300, 699, 700)  # (more than the key-split kernel takes)
    assert "halves" in pick(1, 1400, 1400, 1400) and "halves" not in pick(1, 1399, 1399, 1399)


def test_the_choice_follows_the_number_of_tokens():
    """The same maxima with other totals are other calls (the last answer of a thread is kept by all that the choice depends on)."""
    for _ in range(2):
        assert "halves" in _selected(8, 1000, 1000, 600)
        assert "halves" not in _selected(8, 1000, 1000, 8000)


def test_answers_are_kept_over_other_numbers_of_tokens():
    """Calls with the same maxima are looked up anew (a line of the log) only when their tiles come to lie between other whole numbers
    of tiles per compute unit."""
    code = """import sys
sys.path.insert(0, 'tests')
from test_prefill_halves import _selected
for total in list(range(3700, 4500, 7)) + [8000] + list(range(3700, 4500, 7)):  # 4 to 5 tiles per compute unit, 8, 4 to 5
    _selected(16, 1000, 1000, total)
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), env=dict(os.environ, ATTN_LOG="1"),
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert sum(l.startswith("[attn] prefill") for l in r.stderr.splitlines()) == 3


@pytest.mark.gpu
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n", [40, 97, 300])
def test_infinite_values_reach_the_same_rows(d, n):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").to(torch.bfloat16) for h in (8, 2, 2))
    for key in (0, n // 2, n - 1):
        v[key, key % 2, 5] = math.inf
    starts = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    lens = torch.tensor([n], dtype=torch.int32, device="cuda")
    got = []
    try:
        for kind in ("w4 hpw4 slots4 pf4 seqmajor", "w8 hpw4 slots4 pf4 halves seqmajor"):
            name = "prefill_bf16_ring d%d qb1 %s" % (d, kind)
            ids = [i for i in range(A.attn_num_instances(False)) if A.attn_instance_name(False, i) == name]
            A.attn_force_instance(False, ids[0])
            out = torch.empty_like(q)
            A.attn_prefill_varlen(q, k, v, out, starts, lens, 1.0 / math.sqrt(d), max_q_len=n, max_kv_len=n)
            got.append(out.float().cpu())
    finally:
        A.attn_force_instance(False, -1)
    one, two = got
    assert not torch.isfinite(one).all()
    # (a row that sees an infinity is infinite or NaN, by whether the key's unit hides others from it: the same units in both)
    assert torch.equal(torch.isnan(one), torch.isnan(two)) and torch.equal(torch.isposinf(one), torch.isposinf(two))
