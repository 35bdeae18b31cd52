"""The addresses that the products fetch from straight into LDS, and the bf16 ReLU mask of every value, checked on the host
(async_bounds.hip)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_addresses_stay_inside_their_arrays(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "async_bounds")
    subprocess.check_call([hipcc, "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-function",
                           "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_2305_09887_amd", "csrc"), os.path.join(HERE, "async_bounds.hip"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
