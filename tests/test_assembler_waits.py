"""Distances that the hardware does not keep and the compiler keeps only between instructions that it knows, so not from or to
those written in assembler: two wait states from a vector instruction to a matrix instruction that reads its result, five from
a vector instruction that writes a scalar register to a memory instruction that reads it.  Read from the assembly of products
whose operands are fetched in assembler (assembler_waits.hip)."""
import os
import re
import subprocess

import pytest

from paper_2305_09887_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def registers(text, kind):
    found = set()
    for m in re.finditer(r"(?<![a-z0-9_])" + kind + r"(?:(\d+)|\[(\d+):(\d+)\])", text):
        found.update(range(int(m[1] or m[2]), int(m[1] or m[3]) + 1))
    return found


def too_near(assembly):
    """The instructions of `assembly` that come too early, and how many were looked at: fetches and matrix instructions."""
    wrong, fetches, products = [], 0, 0
    by_hand, now, vector, scalar, kernel = False, 0, {}, {}, ""     # registers: when they were written
    for line in assembly.splitlines():
        if line.startswith("_Z"):
            vector, scalar, kernel = {}, {}, line.split(":")[0]
        line = line.strip()
        if line.startswith(";;#ASM"):
            by_hand = line == ";;#ASMSTART"
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        out, _, read = rest.partition(",")
        if op.startswith("v_mfma"):
            products += 1
            wrong += [(kernel, line) for r in registers(read, "v") if now - vector.get(r, -9) <= 2]
        elif op.startswith("global_load_lds") and by_hand:
            fetches += 1
            wrong += [(kernel, line) for r in registers(rest, "s") if now - scalar.get(r, -9) <= 5]
        elif op.startswith("v_"):
            for r in registers(out, "v"):
                vector.pop(r, None)
                if by_hand:
                    vector[r] = now
            carry = read.split(",")[0] if "_co_" in op else ""
            scalar.update({r: now for r in registers(out + " " + carry, "s")})
        elif op.startswith("s_"):
            for r in registers(out, "s"):
                scalar.pop(r, None)
        now += 1 + (int(rest, 0) if op == "s_nop" else 0)
    return wrong, fetches, products


def test_a_planted_one_is_seen():
    near = ";;#ASMSTART\nv_pk_mul_lo_u16 v3, v4, v5\n;;#ASMEND\ns_nop 0\nv_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[24:27], v[8:23]\n"
    assert len(too_near(near)[0]) == 1
    assert not too_near(near.replace("s_nop 0", "s_nop 1"))[0]
    load = "v_readfirstlane_b32 s4, v0\n;;#ASMSTART\ns_mov_b32 m0, s9\ns_nop 0\nglobal_load_lds_dwordx4 v1, s[4:5]\n;;#ASMEND\n"
    assert len(too_near(load)[0]) == 1
    assert not too_near(load.replace("s_nop 0", "s_nop 3"))[0]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("waits") / "device.s"
    subprocess.check_call([build.HIPCC, *build.FLAGS, "-Wno-unused-function", "--offload-device-only", "-S", os.path.join(HERE, "assembler_waits.hip"), "-o", str(out)])
    return out.read_text()


def test_distances(assembly):
    wrong, fetches, products = too_near(assembly)
    assert fetches > 50 and products > 50
    assert not wrong, wrong[:5]


def test_the_compiler_knows_what_a_fetch_writes(assembly):
    """Where a fetch goes is in m0: its own loads into LDS around one by hand have it set again."""
    kernel = assembly[assembly.index("two_ways"):]
    kernel = kernel[kernel.index("two_ways"):kernel.index("s_endpgm")]
    steps = re.findall(r"s_mov_b32 m0|global_load_lds_dword", kernel)
    assert steps == ["s_mov_b32 m0", "global_load_lds_dword"] * 3, steps
