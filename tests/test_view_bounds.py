"""The operand views of the products never read outside their arrays: run on the host, over every position of every tile,
on arrays between unreadable pages (view_bounds.hip).  Widths of every remainder of four and eight, rows with and without
padding, down to one row and one column."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("views") / "view_bounds")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    subprocess.check_call([hipcc, "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-function",
                           "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_2305_09887_amd", "csrc"), os.path.join(HERE, "view_bounds.hip"), "-o", exe])
    return exe


@pytest.mark.parametrize("F_in,F_out,n", [(1, 1, 1), (1, 4, 1), (4, 1, 1), (2, 2, 1), (7, 3, 1), (1, 5, 2), (3, 2, 2), (5, 300, 2),
                                          (63, 20, 5), (62, 21, 3), (61, 19, 4), (64, 12, 33), (150, 41, 7), (90, 150, 17),
                                          (59, 28, 130), (103, 36, 6), (128, 47, 31)])
def test_views_stay_inside_their_arrays(program, F_in, F_out, n):
    r = subprocess.run([program, str(F_in), str(F_out), str(n)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, f"ended with {r.returncode} at: {r.stdout.splitlines()[-1]}"
