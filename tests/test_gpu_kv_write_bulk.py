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


def _padded(tokens, live):
    H, D, bs = 8, 128, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(tokens + live)
    k, v = (torch.randn(tokens, H, D, generator=g, device="cuda").bfloat16() for _ in range(2))
    slots = torch.randperm(tokens, generator=g, device="cuda").int()
    slots[live:] = -1
    return k, v, [torch.zeros(tokens // bs, bs, H, D, dtype=torch.bfloat16, device="cuda") for _ in range(2)], slots


@pytest.mark.parametrize("live", [0, 1, 4, 4094, 8189])
def test_bulk_write_padded_at_the_end(live):
    k, v, caches, slots = _padded(8192, live)
    A.attn_kv_cache_write(k, v, *caches, slots)
    for cache, new in zip(caches, (k, v)):
        want = torch.zeros_like(cache).view(8192, 8, 128)
        want[slots[:live].long()] = new[:live]
        assert torch.equal(cache.view(8192, 8, 128), want)


def test_padding_costs_no_traffic():
    """16384 tokens of which 400 are real: the rest is skipped, not read (0.17 of a full call's time; read but not stored, 0.46)."""
    def us(live):
        sets = [_padded(16384, live) for _ in range(3)]
        for x in sets:
            A.attn_kv_cache_write(x[0], x[1], *x[2], x[3])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()  # (eager calls are bound by the host)
        with torch.cuda.graph(graph):
            for k, v, c, s in sets * 4:
                A.attn_kv_cache_write(k, v, *c, s)
        times = []
        for _ in range(20):
            e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
            e0.record()
            graph.replay()
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1) * 1000 / 12)
        return sorted(times)[10]

    full, padded = us(16384), us(400)
    print("full %.1f us, padded %.1f us" % (full, padded), flush=True)
    assert padded <= 0.33 * full
