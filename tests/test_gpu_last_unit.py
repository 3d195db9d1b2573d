"""The ring prefill kernels' scores stay one fused multiply-add from the exponential wherever a unit of 32 keys hides nothing, in the
last unit of a tile, of a part and of a half of the keys too.  Scores near 2^23, a few apart: scaled and rounded to 32 bits first they
would be off by up to 1/16 in the exponent, 4 % of a weight."""
import numpy as np
import pytest
import torch

import paper_2505_03780_amd as A

pytestmark = pytest.mark.gpu

SCALE = float(np.float32(0.1))
TYPES = {"bf16": (torch.bfloat16, 2.0 ** -8), "f16": (torch.float16, 2.0 ** -11)}


def _problem(D, dtype, n_q, n_kv, unit):
    """Queries that see scores 2^23 + (0..31) in `unit`, 96 less in the others (a weight of 1e-4), and the exact result."""
    g = torch.Generator().manual_seed(n_kv + unit)
    q, k = torch.zeros(n_q, 4, D), torch.zeros(n_kv, 1, D)
    q[..., 0], q[..., 1] = 4096.0, 1.0
    k[:, 0, 0] = 2048.0
    j = torch.arange(n_kv)
    k[:, 0, 1] = (j % 32 - torch.where(j // 32 == unit, 0, 96)).float()
    v = torch.randn(n_kv, 1, D, generator=g).to(TYPES[dtype][0]).double()
    w = torch.softmax(k[:, 0, 1].double() * SCALE, 0)
    ref, spread = w @ v[:, 0], w @ v[:, 0].abs()
    # rounding of every weight and of the result, and the smallest difference of two scaled scores in 32 bits
    bound = TYPES[dtype][1] * (spread + ref.abs()) * 1.01 + 1e-4
    dev = lambda t: t.to(TYPES[dtype][0]).cuda()
    return dev(q), dev(k), dev(v), ref, bound


def _call(q, k, v, causal, workspace=None):
    n_q, n_kv = q.shape[0], k.shape[0]
    ints = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")
    out = torch.empty_like(q)
    A.attn_prefill_varlen(q, k, v, out, ints(0, n_q), ints(n_kv), SCALE, max_q_len=n_q, max_kv_len=n_kv, causal=causal, kv_start_loc=ints(0, n_kv),
                          workspace=workspace)
    return out.double().cpu()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("n_units", [1, 2, 5, 10, 18])
def test_a_whole_last_unit_is_as_exact_as_any(D, dtype, n_units):
    done = 0
    for unit in sorted({n_units - 1, (n_units + 1) // 2 - 1, 0}):  # the last one, the last of the first half
        q, k, v, ref, bound = _problem(D, dtype, 40, 32 * n_units, unit)
        try:
            for i in range(A.attn_num_instances(False)):
                name = A.attn_instance_name(False, i)
                if "prefill_%s_ring d%d " % (dtype, D) not in name or "hpw8" in name:
                    continue
                A.attn_force_instance(False, i)
                print(name, flush=True)
                off = (_call(q, k, v, False) - ref).abs()
                assert (off <= bound).all(), (name, unit, (off / bound).max())
                done += 1
        finally:
            A.attn_force_instance(False, -1)
    assert done >= 12


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("D", [128, 64])
def test_the_last_unit_of_a_part(D, dtype):
    n_kv, n_q = 4096, 33
    q, k, v, _, _ = _problem(D, dtype, n_q, n_kv, 0)
    try:
        name = "prefill_%s_ring d%d qb1 w4 hpw4 slots4 pf4 seqmajor" % (dtype, D)
        A.attn_force_instance(False, [A.attn_instance_name(False, i) for i in range(A.attn_num_instances(False))].index(name))
        ints = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")
        a = A.make_args(q, k, v, torch.empty_like(q), ints(n_kv), SCALE, max_q_len=n_q, max_kv_len=n_kv, query_start_loc=ints(0, n_q),
                        kv_start_loc=ints(0, n_kv), causal=True)
        parts = A.attn_prefill_parts_instance(a)[1]
        assert parts > 1
        length = -(-(-(-n_kv // parts)) // 256) * 256
        scratch = torch.empty(A.attn_prefill_scratch_bytes(a), dtype=torch.uint8, device="cuda")
        for end in (length, 2 * length, 32):
            q, k, v, ref, bound = _problem(D, dtype, n_q, n_kv, end // 32 - 1)
            off = (_call(q, k, v, True, scratch) - ref).abs()
            assert (off <= bound).all(), (name, end, (off / bound).max())
    finally:
        A.attn_force_instance(False, -1)
