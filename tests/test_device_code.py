"""Properties of the generated gfx950 code (CPU: compiled here, read as assembly)."""
import os
import re
import subprocess

import pytest

from paper_1506_06513_amd.build import CSRC, HIPCC_FLAGS, hipcc


def _asm(tmp_path, text):
    src = os.path.join(tmp_path, "unit.hip")
    with open(src, "w") as f:
        f.write(f'#include "{os.path.join(CSRC, "kernels.hpp")}"\n{text}\n')
    out = os.path.join(tmp_path, "unit.s")
    subprocess.run([hipcc(), *HIPCC_FLAGS, "-S", "--offload-device-only", src, "-o", out], check=True,
                   capture_output=True, timeout=300)
    return open(out).read()


def _body(asm, name):
    """Instructions of the kernel whose mangled name contains `name`."""
    m = re.search(r"^(_ZN\S*" + name + r"\S*):.*?\n(.*?)^\s*s_endpgm", asm, re.M | re.S)
    assert m, name
    return [ln.split(";")[0].strip() for ln in m.group(2).splitlines()]


def _foreign_scalar_loads(ins):
    """Scalar loads from anything but the kernel arguments (s[0:1] on entry) and
    constants of the code object (s_getpc)."""
    known, out = {"s[0:1]"}, []
    for line in ins:
        op, _, rest = line.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op == "s_mov_b64" and args[1] in known:
            known.add(args[0])
        elif op == "s_getpc_b64":
            known.add(args[0])
        elif op.startswith("s_load_") and args[1] not in known:
            out.append(line)
    return out


@pytest.mark.parametrize("real", ["float", "double"])
def test_prologue_reads_no_memory_through_the_scalar_cache(tmp_path, real):
    # the prologue writes the launch record by vector stores and works on it: scalar
    # loads of it would not wait for these stores and could return another record
    asm = _asm(tmp_path, f"namespace flusi {{ template __global__ void k_prologue<{real}>(Member*, long, Member, "
                         "flusi_insect); }")
    assert _foreign_scalar_loads(_body(asm, "k_prologue")) == []


@pytest.mark.parametrize("n", [128, 256])
def test_forward_real_transform_leaves_room_for_five_waves(tmp_path, n):
    # 512 vector registers per lane and SIMD, in steps of 8: five waves take 96 at most
    asm = _asm(tmp_path, f"namespace flusi {{ template __global__ void k_x_r2c<double, {n}>(const double*, "
                         "cx<double>*, long, int, int, const cx<double>*); }")
    meta = asm[asm.index(".amdgpu_metadata"):]
    entry = next(e for e in meta.split("  - .agpr_count") if "k_x_r2c" in e)
    assert int(re.search(r"\.vgpr_count:\s+(\d+)", entry).group(1)) <= 96
    assert int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry).group(1)) == 0


def test_no_rounding_is_left_to_the_code_around_an_expression(tmp_path):
    # an operation flagged "contract" may or may not join an FMA, by its context: tile
    # variants and launch forms of one pass would then differ in the last bit
    out = os.path.join(tmp_path, "unit.ll")
    subprocess.run([hipcc(), *HIPCC_FLAGS, "-DFLUSI_N=16", "-S", "-emit-llvm", "--offload-device-only",
                    os.path.join(CSRC, "inst.hip"), "-o", out], check=True, capture_output=True, timeout=300)
    flagged = [ln.strip() for ln in open(out) if re.search(r"= f(add|sub|mul) (\w+ )*contract ", ln)]
    assert flagged == []
