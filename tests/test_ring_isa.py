"""Static hazard check of the ring prefill kernels (see ring_isa_lint.py): no instruction may touch a
register while one of the loop's untracked LDS reads, or its untracked scalar load, may still be in
flight into it.  Runs on the CPU: hipcc cross-compiles the two translation units to assembly."""
import concurrent.futures as cf
import os
import subprocess

import paper_2505_03780_amd as A
import ring_isa_lint as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_03780_amd", "csrc")


def _asm(src, out):
    from paper_2505_03780_amd import build as B

    cmd = ["hipcc", *B.FLAGS, *B.EXTRA.get(src, []), "-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", out]
    subprocess.check_call(cmd, stderr=subprocess.DEVNULL)
    return open(out).read()


def test_no_register_is_touched_while_an_untracked_load_may_land_in_it(tmp_path):
    srcs = ["prefill_bf16_ring.hip", "prefill_f16_ring.hip"]
    with cf.ThreadPoolExecutor(max_workers=2) as ex:
        texts = list(ex.map(lambda s: _asm(s, str(tmp_path / s.replace(".hip", ".s"))), srcs))
    seen = 0
    for text in texts:
        for name, body in L.kernels(text):
            if "prefill_ring_kernel" not in name:
                continue
            seen += 1
            assert any(l.startswith("ds_read_b64_tr_b16") for l in body), name  # the kernel the check is about
            problems = L.lint(body)
            assert not problems, (name, problems[:5])
    # every instance paged and packed (both grid orders are one kernel), the small workgroups also in parts
    names = {A.attn_instance_name(False, i).replace(" seqmajor", "") for i in range(A.attn_num_instances(False))}
    assert seen == sum(4 if " qb1 w4 " in n else 2 for n in names if "_ring " in n)


def test_the_check_sees_a_planted_hazard():
    body = ["s_waitcnt lgkmcnt(0)", ";;#ASMSTART", "ds_read_b128 v[4:7], v1 offset:0", ";;#ASMEND", "ds_read_b128 v[8:11], v1 offset:16",
            "s_waitcnt lgkmcnt(1)", "v_add_f32_e32 v0, v4, v5", "v_mov_b32_e32 v9, 0", "s_waitcnt lgkmcnt(0)", "v_add_f32_e32 v0, v8, v9"]
    problems = L.lint(body)
    assert [p[0] for p in problems] == [7]  # only the write into v9 while the second read is in flight
    loop = [".LBB0_1:", "v_add_f32_e32 v0, v4, v4", "ds_read_b128 v[4:7], v1 offset:0", "s_cbranch_scc1 .LBB0_1", "s_waitcnt lgkmcnt(0)", "s_endpgm"]
    problems = L.lint(loop)
    # seen on the second trip: the read of the previous trip is still in flight when v4 is used and when it is loaded again
    assert [p[0] for p in problems] == [1, 2]
    # the wait stands on one of two paths only
    skipped = ["ds_read_b128 v[4:7], v1 offset:0", "s_cbranch_scc1 .LBB0_1", "s_waitcnt lgkmcnt(0)", ".LBB0_1:", "v_add_f32_e32 v0, v4, v5", "s_endpgm"]
    assert [p[0] for p in L.lint(skipped)] == [4]
    # ... and on both, by way of a block further down
    both = ["s_load_dword s4, s[0:1], 0x0", "s_cbranch_scc1 .LBB0_2", "s_waitcnt lgkmcnt(0)", ".LBB0_1:", "s_add_i32 s5, s4, 1", "s_endpgm", ".LBB0_2:",
            "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_branch .LBB0_1"]
    assert L.lint(both) == []
    both[7] = "s_waitcnt vmcnt(0) lgkmcnt(1)"
    assert [p[0] for p in L.lint(both)] == [4]
