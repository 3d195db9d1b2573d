"""Performance cases of the library: the calls that an LLM inference engine makes through the package's
public entry points, with inputs made on the GPU from a seed.

A case is a dict of plain values.  Its lengths are drawn from `len_seed` (and the bounds next to it), so that
the work of a case does not depend on the seed of its contents; queries, keys, values, activations, block
tables and slot mappings come from the seed given to prepare().  The bounds and the length seeds of the
listed attention cases are those of the benchmark configurations in workloads.py where one fits.

Kinds:
  prefill  attn_prefill_varlen over packed keys (`block` 0) or, through the block table, over a paged cache
           with a cached prefix of `plo`..`phi` keys in front of the `lo`..`hi` new tokens of each sequence
  decode   attn_decode_paged: one query token per sequence, contexts of `lo`..`hi` keys
  rmsnorm  rmsnorm_fused_add, the residual stream updated in place
  kvwrite  attn_kv_cache_write of one step's new keys and values
"""
import math

import numpy as np
import torch

import paper_2505_03780_amd as A

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
SIZE = {"bf16": 2, "f16": 2, "f32": 4}


def _prefill(name, len_seed, batch, lo, hi, hq, hkv, d, dtype, block=0, plo=0, phi=0, causal=True):
    c = {"kind": "prefill", "len_seed": len_seed, "batch": batch, "lo": lo, "hi": hi, "plo": plo, "phi": phi,
         "hq": hq, "hkv": hkv, "d": d, "dtype": dtype, "block": block, "causal": causal}
    return dict(c, name=name) if name else c


def _decode(name, len_seed, batch, lo, hi, hq, hkv, d, dtype, block):
    c = {"kind": "decode", "len_seed": len_seed, "batch": batch, "lo": lo, "hi": hi, "hq": hq, "hkv": hkv, "d": d,
         "dtype": dtype, "block": block}
    return dict(c, name=name) if name else c


def _rmsnorm(name, tokens, hidden, dtype, residual):
    c = {"kind": "rmsnorm", "tokens": tokens, "hidden": hidden, "dtype": dtype, "residual": residual}
    return dict(c, name=name) if name else c


def _kvwrite(name, tokens, hkv, d, dtype, block):
    c = {"kind": "kvwrite", "tokens": tokens, "hkv": hkv, "d": d, "dtype": dtype, "block": block}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small model's prompt in fp32, as in a numerics check or an embedding call: latency
        _prefill("prefill_f32_tiny", 1, 1, 128, 128, 4, 4, 64, "f32"),
        # a prompt batch of a server, lengths mixed (benchmark configuration 3)
        _prefill("prefill_bf16_batch", 3, 8, 256, 2048, 32, 8, 128, "bf16"),
        # one long document, an odd number of tokens
        _prefill("prefill_bf16_long", 6, 1, 8191, 8191, 32, 8, 128, "bf16"),
        # head size 64 (the smaller models' head), fp16, mixed lengths
        _prefill("prefill_f16_d64", 7, 6, 300, 3000, 32, 8, 64, "f16"),
        # chunked prefill: 512 new tokens behind a cached prefix (benchmark configuration 4)
        _prefill("chunk_bf16_batch", 4, 16, 512, 512, 32, 8, 128, "bf16", block=16, plo=0, phi=8192),
        # the next turn of a few chats: some dozens of new tokens behind a long cached history
        _prefill("chunk_bf16_turn", 8, 3, 17, 70, 32, 8, 128, "bf16", block=16, plo=5000, phi=9000),
        # one user's token: the smallest decode call
        _decode("decode_bf16_one", 9, 1, 1900, 1900, 32, 8, 128, "bf16", 16),
        # a decode step of a full batch (benchmark configuration 2)
        _decode("decode_bf16_batch", 2, 64, 512, 4096, 32, 8, 128, "bf16", 16),
        # long contexts, 64 query heads (benchmark configuration 5)
        _decode("decode_bf16_long", 5, 16, 16384, 32768, 64, 8, 128, "bf16", 16),
        # many short chats in fp16, another block size
        _decode("decode_f16_short", 10, 200, 20, 800, 32, 8, 128, "f16", 32),
        # the layer norm in front of attention for a prompt batch
        _rmsnorm("rmsnorm_bf16", 8192, 4096, "bf16", True),
        # the keys and values of a prompt batch stored into the paged cache
        _kvwrite("kvwrite_bf16", 8192, 8, 128, "bf16", 16),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


HEADS = [(32, 8), (32, 8), (64, 8), (8, 2), (16, 16), (16, 4)]


def draw(rng):
    """One more case of the same ranges, at most about as costly as the largest listed one of its kind."""
    while True:
        seed = rng.randrange(1 << 20)
        kind = rng.choice(["prefill", "prefill", "chunk", "chunk", "decode", "decode", "decode", "f32", "rmsnorm", "kvwrite"])
        hq, hkv = rng.choice(HEADS)
        dtype = rng.choice(["bf16", "bf16", "f16"])
        block = rng.choice([16, 16, 32, 64, 128])
        if kind == "prefill":
            hi = _log(rng, 16, 8192)
            c = _prefill(None, seed, _log(rng, 1, 64), max(1, hi // rng.randint(1, 8)), hi, hq, hkv, rng.choice([128, 128, 64]), dtype,
                         block=rng.choice([0, 0, block]), causal=rng.random() < 0.85)
            if work(c)["flops"] > (100e9 if c["d"] == 64 else 500e9):
                continue
        elif kind == "chunk":
            phi = _log(rng, 64, 16384)
            hi = _log(rng, 1, 1024)
            c = _prefill(None, seed, _log(rng, 1, 32), max(1, hi // rng.randint(1, 4)), hi, hq, hkv, rng.choice([128, 128, 128, 64]), dtype,
                         block=block, plo=phi // rng.randint(1, 8), phi=phi)
            if work(c)["flops"] > (100e9 if c["d"] == 64 else 500e9):
                continue
        elif kind == "decode":
            hi = _log(rng, 16, 32768)
            c = _decode(None, seed, _log(rng, 1, 256), max(1, hi // rng.randint(1, 8)), hi, hq, hkv, rng.choice([128, 128, 128, 64]), dtype, block)
            if work(c)["bytes"] > 1.6e9:
                continue
        elif kind == "f32":
            hi = _log(rng, 16, 512)
            hq, hkv = rng.choice([(4, 4), (8, 2), (8, 8)])
            c = _prefill(None, seed, _log(rng, 1, 4), max(1, hi // rng.randint(1, 4)), hi, hq, hkv, rng.choice([64, 64, 128]), "f32",
                         block=rng.choice([0, 0, 16]))
        elif kind == "rmsnorm":
            c = _rmsnorm(None, _log(rng, 1, 16384), rng.choice([1024, 2048, 2560, 3072, 4096, 5120, 8192]), dtype, rng.random() < 0.75)
            if work(c)["bytes"] > 600e6:
                continue
        else:
            c = _kvwrite(None, _log(rng, 1, 16384), hkv, rng.choice([128, 64]), dtype, block)
        return c


def _lengths(case):
    """(new tokens, keys) of every sequence of an attention case."""
    rng = np.random.default_rng(case["len_seed"])
    n = case["batch"]
    if case["kind"] == "decode":
        return np.ones(n, np.int64), rng.integers(case["lo"], case["hi"], size=n, endpoint=True)
    if case["block"] == 0 or case["phi"] == 0:
        new = rng.integers(case["lo"], case["hi"], size=n, endpoint=True)
        return new, new.copy()
    prefix = rng.integers(case["plo"], case["phi"], size=n, endpoint=True)
    new = rng.integers(case["lo"], case["hi"], size=n, endpoint=True)
    return new, prefix + new


def work(case):
    if case["kind"] == "rmsnorm":
        n = case["tokens"] * case["hidden"]
        return {"bytes": 2.0 * n * (4 if case["residual"] else 2) + 2 * case["hidden"], "flops": 5.0 * n}
    if case["kind"] == "kvwrite":
        return {"bytes": 4.0 * case["tokens"] * case["hkv"] * case["d"] * SIZE[case["dtype"]] + 4 * case["tokens"], "flops": 0.0}
    new, keys = _lengths(case)
    if case.get("causal", True):
        pairs = int(np.sum(new * (keys - new) + new * (new + 1) // 2))
    else:
        pairs = int(np.sum(new * keys))
    size = SIZE[case["dtype"]]
    data = int(keys.sum()) * case["hkv"] * case["d"] * 2 * size + 2 * int(new.sum()) * case["hq"] * case["d"] * size
    table = 4 * int(np.sum(-(-keys // case["block"]))) if case["block"] else 0
    return {"bytes": float(data + table), "flops": 4.0 * case["d"] * case["hq"] * pairs}


def tolerance(case):
    if case["kind"] == "kvwrite":
        return "exact"
    if case["kind"] == "rmsnorm":
        # one rounding of each output: half an ulp is at most 2^-8 (bf16) or 2^-11 (fp16) of a value, and sums
        # in another order move a value across a rounding boundary now and then, by a whole ulp
        return {"rel": 1e-3, "max": 1.6e-2} if case["dtype"] == "bf16" else {"rel": 1.3e-4, "max": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 5e-5}
    return {"rel": 8e-3, "max": 6e-2} if case["dtype"] == "bf16" else {"rel": 1e-3, "max": 1e-2}


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, scale=1.0, shift=0.0):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    for lo in range(0, flat.numel(), 1 << 26):
        part = flat[lo:lo + (1 << 26)]
        part.copy_(torch.randn(part.numel(), generator=g, device="cuda") * scale + shift)
    return out


def _int32(values):
    return torch.from_numpy(np.ascontiguousarray(values, dtype=np.int32)).cuda()


def _starts(lens):
    return np.concatenate([[0], np.cumsum(lens)])


def _attention_inputs(case, seed):
    """Queries, keys and values, lengths on the host and on the GPU, and for a paged case the block table: every
    sequence takes the next blocks of a random permutation of the pool, unused entries are -1."""
    g = _generator(seed)
    new, keys = _lengths(case)
    dtype, hq, hkv, d, block = DTYPES[case["dtype"]], case["hq"], case["hkv"], case["d"], case["block"]
    s = {"new": new, "keys": keys, "q": _normal(g, (int(new.sum()), hq, d), dtype)}
    if block:
        need = -(-keys // block)
        blocks = int(need.sum()) + 7
        perm = np.random.default_rng(seed).permutation(blocks)
        table = np.full((len(keys), int(need.max())), -1, np.int64)
        at = 0
        for i, n in enumerate(need):
            table[i, :n] = perm[at:at + n]
            at += int(n)
        s["table_host"], s["table"] = table, _int32(table)
        shape = (blocks, block, hkv, d)
    else:
        s["table_host"], s["table"] = None, None
        shape = (int(keys.sum()), hkv, d)
    s["k"] = _normal(g, shape, dtype)
    s["v"] = _normal(g, shape, dtype)
    s["scale"] = 1.0 / math.sqrt(d)
    s["keys_gpu"], s["starts_gpu"] = _int32(keys), _int32(_starts(new))
    return s


def prepare(case, seed):
    if case["kind"] == "rmsnorm":
        g, dtype, shape = _generator(seed), DTYPES[case["dtype"]], (case["tokens"], case["hidden"])
        s = {"x": _normal(g, shape, dtype), "weight": _normal(g, shape[1:], dtype, 0.1, 1.0), "eps": 1e-5,
             "residual": _normal(g, shape, dtype, 2.0) if case["residual"] else None}
        s["out"] = torch.empty_like(s["x"])
        return dict(s, case=case)
    if case["kind"] == "kvwrite":
        g, dtype = _generator(seed), DTYPES[case["dtype"]]
        tokens, block = case["tokens"], case["block"]
        blocks = -(-tokens // block) + 64
        rng = np.random.default_rng(seed)
        # prompts fill whole blocks, taken from the pool in random order; one token in 64 is padding
        blocks_of = rng.permutation(blocks)[:-(-tokens // block)]
        slots = (blocks_of[:, None] * block + np.arange(block)[None, :]).reshape(-1)[:tokens]
        slots[rng.random(tokens) < 1.0 / 64] = -1
        shape = (tokens, case["hkv"], case["d"])
        cache = (blocks, block, case["hkv"], case["d"])
        return {"k": _normal(g, shape, dtype), "v": _normal(g, shape, dtype), "k_cache": torch.zeros(cache, dtype=dtype, device="cuda"),
                "v_cache": torch.zeros(cache, dtype=dtype, device="cuda"), "slots": _int32(slots), "case": case}
    s = _attention_inputs(case, seed)
    s["out"] = torch.empty_like(s["q"])
    s["max_new"], s["max_keys"] = int(s["new"].max()), int(s["keys"].max())
    if case["kind"] == "decode":
        args = A.make_args(s["q"], s["k"], s["v"], s["out"], s["keys_gpu"], s["scale"], max_q_len=1, max_kv_len=s["max_keys"],
                           block_table=s["table"], is_decode=True)
        s["workspace"] = torch.empty(max(16, A.attn_workspace_bytes(args, True)), dtype=torch.uint8, device="cuda")
    return dict(s, case=case)


def run(s):
    kind = s["case"]["kind"]
    if kind == "prefill":
        A.attn_prefill_varlen(s["q"], s["k"], s["v"], s["out"], s["starts_gpu"], s["keys_gpu"], s["scale"], max_q_len=s["max_new"],
                              max_kv_len=s["max_keys"], causal=s["case"]["causal"], block_table=s["table"])
        return s["out"]
    if kind == "decode":
        A.attn_decode_paged(s["q"], s["k"], s["v"], s["out"], s["table"], s["keys_gpu"], s["scale"], max_kv_len=s["max_keys"],
                            workspace=s["workspace"])
        return s["out"]
    if kind == "rmsnorm":
        A.rmsnorm_fused_add(s["x"], s["weight"], s["out"], s["eps"], residual=s["residual"])
        return {"out": s["out"], "residual": s["residual"]} if s["residual"] is not None else {"out": s["out"]}
    A.attn_kv_cache_write(s["k"], s["v"], s["k_cache"], s["v_cache"], s["slots"])
    return {"k_cache": s["k_cache"], "v_cache": s["v_cache"]}


def exact(case, seed):
    if case["kind"] == "kvwrite":
        return None
    if case["kind"] == "rmsnorm":
        s = prepare(case, seed)
        z = s["x"].double()
        if s["residual"] is not None:
            z = z + s["residual"].double()
        out = z / torch.sqrt((z * z).mean(dim=1, keepdim=True) + s["eps"]) * s["weight"].double()
        return {"out": out, "residual": z} if s["residual"] is not None else {"out": out}
    s = _attention_inputs(case, seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    group = hq // hkv
    out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
    starts, kstarts = _starts(s["new"]), _starts(s["keys"])
    causal = case.get("causal", True)
    for i, (n, m) in enumerate(zip(s["new"], s["keys"])):
        n, m = int(n), int(m)
        if case["block"]:
            rows = s["table"][i, :-(-m // case["block"])].long()
            k, v = (s[x][rows].reshape(-1, hkv, d)[:m].double() for x in ("k", "v"))
        else:
            k, v = (s[x][int(kstarts[i]):int(kstarts[i]) + m].double() for x in ("k", "v"))
        q = s["q"][int(starts[i]):int(starts[i]) + n].double()
        for h in range(hkv):
            kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
            for a in range(0, n, 1024):
                b = min(n, a + 1024)
                scores = (q[a:b, h * group:(h + 1) * group].reshape(-1, d) @ kt) * s["scale"]
                if causal and n > 1:
                    last = torch.arange(m - n + a, m - n + b, device="cuda").repeat_interleave(group)
                    scores.masked_fill_(torch.arange(m, device="cuda")[None, :] > last[:, None], -math.inf)
                out[int(starts[i]) + a:int(starts[i]) + b, h * group:(h + 1) * group] = (torch.softmax(scores, dim=1) @ vh).reshape(b - a, group, d)
    return out
