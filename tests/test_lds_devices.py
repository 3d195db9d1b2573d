"""Kernels that take more than 64 KB of LDS ask for it on every device that they are launched on, not on the first alone
(tests/lds_devices.cpp; the HIP runtime's calls are replaced by the program's own, no GPU)."""
import os
import subprocess

import paper_2505_03780_amd as A

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2505_03780_amd")


def test_every_device_is_asked(tmp_path):
    A.load_library()
    exe = str(tmp_path / "lds_devices")
    subprocess.check_call(["g++", "-O1", "-rdynamic", os.path.join(ROOT, "tests", "lds_devices.cpp"), "-o", exe, "-L" + PKG, "-lattn_gfx950", "-Wl,-rpath," + PKG,
                           "-Wl,--unresolved-symbols=ignore-in-shared-libs"])
    env = {k: v for k, v in os.environ.items() if not k.startswith("ATTN_") and k != "LD_PRELOAD"}
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
