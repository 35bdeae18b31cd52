"""Wait states between vector instructions, which the hardware does not keep and the compiler keeps only between instructions that it knows: two from one that writes
a scalar register to one that reads it (the carry of a 64-bit addition is one), and from one that writes a vector register to one that reads it from another
lane.  Read from the assembly of the gathers, whose lanes add what others multiplied, and of the products whose operands are fetched in assembler."""
import os
import re
import subprocess

import pytest

from paper_2305_09887_amd import build
from test_assembler_waits import HERE, registers


def scalars(text):
    return registers(text, "s") | ({"vcc"} if "vcc" in text else set())


def too_near(assembly):
    """The instructions of `assembly` that come too early, and how many of the two kinds were looked at."""
    wrong, carries, lanes = [], 0, 0
    now, vector, scalar, kernel = 0, {}, {}, ""     # registers: when they were written
    for line in assembly.splitlines():
        if line.startswith("_Z"):
            vector, scalar, kernel = {}, {}, line.split(":")[0]
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        out, _, read = rest.partition(",")
        if op.startswith("v_") and not op.startswith("v_mfma"):
            carry = ""
            if "_co_" in op or op.startswith(("v_mad_u64", "v_mad_i64", "v_div_scale")):
                carry, _, read = read.partition(",")
            known = scalars(read) & set(scalar)
            carries += len(known)
            wrong += [(kernel, line) for r in known if now - scalar[r] <= 2]
            if re.search(r"\b(quad_perm|row_\w+|wave_\w+):?", read):      # reads its first operand from another lane
                lanes += 1
                wrong += [(kernel, line) for r in registers(read.split(",")[0], "v") if now - vector.get(r, -9) <= 2]
            vector.update({r: now for r in registers(out, "v")})
            scalar.update({r: now for r in scalars(out + " " + carry)})
        elif op.startswith("s_"):
            for r in scalars(out):
                scalar.pop(r, None)
        now += 1 + (int(rest, 0) if op == "s_nop" else 0)
    return wrong, carries, lanes


def test_a_planted_one_is_seen():
    for of in "quad_perm:[1,1,1,1]", "":
        add = f"v_add_co_u32_e32 v0, vcc, v2, v4 {of}\ns_nop 0\nv_addc_co_u32_e32 v1, vcc, v3, v5, vcc {of}\n"
        assert len(too_near(add)[0]) == 1
        assert not too_near(add.replace("s_nop 0", "s_nop 1"))[0]
    lane = "v_mul_lo_u32 v2, v0, v1\ns_nop 0\nv_add_u32_dpp v3, v2, v4 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n"
    assert len(too_near(lane)[0]) == 1
    assert not too_near(lane.replace("s_nop 0", "s_nop 1"))[0]


@pytest.mark.parametrize("source", [os.path.join(build.CSRC, "spmm.hip"), os.path.join(HERE, "assembler_waits.hip")])
def test_distances(source, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "device.s"
    subprocess.check_call([build.HIPCC, *build.FLAGS, "-Wno-unused-function", "--offload-device-only", "-S", source, "-o", str(out)])
    wrong, carries, lanes = too_near(out.read_text())
    assert carries > 50 and (lanes > 50 or "spmm" not in source)
    assert not wrong, wrong[:5]
