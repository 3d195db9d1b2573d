"""Error of the 16-bit prefill kernels at head size 64 against 64 bits: no larger than that of the register-staged kernel, whose
reference is the running maximum of a row.  The inputs are those on which a reference that lags behind it shows most:
a peaked softmax over enough keys that the maximum moves late."""
import numpy as np
import pytest

import paper_2505_03780_amd as A
import workloads as W
from attn_testlib import DeviceWorkload, oracle_problem, to_host_f64

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("scale", [1.0, 4.0])
def test_error_is_no_larger_than_the_staged_kernels(dtype, scale):
    # 256 rows (heads x tokens) over 6000 keys, eight wavefronts with 750 keys each in the key-split kernel
    wl = W.make_paged(97, "prefill", [64], [6000], 4, 4, 64, 16, 380, scale=scale / 8.0)
    if dtype == "f16":
        wl = W.as_f16(wl)
    dw = DeviceWorkload(wl)
    ref = oracle.attention(oracle_problem(wl))
    errors = {"staged": [], "ring": [], "keysplit": []}
    try:
        for i in range(A.attn_num_instances(False)):
            name = A.attn_instance_name(False, i)
            A.attn_force_instance(False, i)
            if " d64 " not in name or A.attn_selected_instance(dw.args(False), False) != i:
                continue
            err = np.linalg.norm(to_host_f64(dw.run(False)) - ref) / np.linalg.norm(ref)
            errors["ring" if "ring" in name else "keysplit" if "keysplit" in name else "staged"].append(err)
    finally:
        A.attn_force_instance(False, -1)
    print(dtype, scale, {k: ["%.4e" % e for e in v] for k, v in errors.items()}, flush=True)
    staged = max(errors["staged"])
    # The weights' roundings of 256 rows x 6000 keys are independent draws: two kernels of equal precision differ by well
    # under 1 % here; a reference that may lag by 2^8 gives 3 to 23 % more.
    assert errors["ring"] and errors["keysplit"]
    assert max(errors["ring"]) <= 1.01 * staged and max(errors["keysplit"]) <= 1.01 * staged
