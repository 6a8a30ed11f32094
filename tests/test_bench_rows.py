"""Rows per x-pass workgroup in the bench's byte model against the kernels' own (CPU)."""
import os
import subprocess

import bench
from paper_1506_06513_amd.build import CSRC, HIPCC_FLAGS, boxes, hipcc, sizes


def test_x_pass_rows_are_the_kernels(tmp_path):
    lines = [f'#include "{os.path.join(CSRC, "kernels.hpp")}"', "using namespace flusi;"]
    for nx, n in [(n, n) for n in sizes()] + boxes():
        for real, cb in (("float", 8), ("double", 16)):
            for v in range(3):
                lines.append(f"static_assert(xpass_wg_rows<{real}, {nx}, {n}>({v}) == {bench.x_wg_rows(nx, n, cb, v)}, "
                             f'"{real} {nx}x{n} variant {v}");')
    src = os.path.join(tmp_path, "rows.hip")
    with open(src, "w") as f:
        f.write("\n".join(lines) + "\n")
    r = subprocess.run([hipcc(), *HIPCC_FLAGS, "-fsyntax-only", "--offload-host-only", src], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]


def test_the_pass_model_counts_the_variants_records():
    n, s = 256, 8
    KP = (n - 1) // 3 + 1
    fields = 9 * n * n * KP * s
    for v, rows in ((0, 8), (1, 16), (2, 4)):
        assert bench.pass_bytes(n, s, False, x_variant=v)["x_pass"] == fields + n * n // rows * 39 * 8
