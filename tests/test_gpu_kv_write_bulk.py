"""The cache write's four-tokens-per-thread kernel: a last group of one to three tokens, padding inside a group, heads and
tokens with gaps between them, against an index copy."""
import pytest
import torch

import paper_2505_03780_amd as A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,dtype,D", [(4096, torch.bfloat16, 128), (4097, torch.bfloat16, 128), (4099, torch.float32, 64),
                                            (8190, torch.float32, 64), (8191, torch.float32, 768)])  # the last: loads with the hint
def test_bulk_write(tokens, dtype, D):
    assert tokens * 8 * D * torch.empty(0, dtype=dtype).element_size() * 2 // 16 >= (1 << 20 if D < 768 else 6 << 20)
    g = torch.Generator(device="cuda")
    g.manual_seed(tokens)
    H, bs, nb = 8, 16, 520
    wide = torch.randn(tokens, H + 1, D + 8, generator=g, device="cuda").to(dtype)  # gaps behind heads and tokens
    new = wide[:, :H, :D]
    new2 = (wide * 2)[:, :H, :D]
    slots = torch.randperm(nb * bs, generator=g, device="cuda")[:tokens].int()
    slots[5::9] = -1
    slots[-1] = -1 if tokens % 2 else int(slots[-1])
    caches = [torch.zeros(nb, bs, H + 2, D, dtype=dtype, device="cuda") for _ in range(2)]
    want = [c.clone() for c in caches]
    A.attn_kv_cache_write(new, new2, caches[0][:, :, :H], caches[1][:, :, :H], slots)
    keep = slots >= 0
    for w, x in zip(want, (new, new2)):
        w.view(nb * bs, H + 2, D)[slots[keep].long(), :H] = x[keep]
    assert torch.equal(caches[0], want[0]) and torch.equal(caches[1], want[1])  # untouched slots and gaps included
