"""The scans write v_med3_u32 as assembly, into which the compiler does not look
for the wait states that a reader of a matrix product's registers needs.  So
its keys have to be results of vector instructions: checked in the assembly of
the kernels, compiled here for gfx950 (no GPU).
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2008_05612_amd import build

KERNELS = """
#include "gemm_blk.h"
#include "gemm_scan.h"
namespace hpmap {
template __global__ void k_scan<1, true, 1, 8, 1, 2>(EnumJob);
template __global__ void k_scan<1, true, 1, 1, 16, 4>(EnumJob);
template __global__ void k_scan<1, false, 1, 1, 16, 4>(EnumJob);
namespace {
template __global__ void k_gemm_wide<1, true, 1>(EnumJob);
}
}
"""


def _registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"v(\d+)", operand)
    return {int(m.group(1))} if m else set()


def test_median_keys_come_from_vector_instructions(tmp_path):
    if not (os.path.exists(build.HIPCC) or shutil.which(build.HIPCC)):
        pytest.skip("no hipcc")
    src, out = tmp_path / "kernels.hip", tmp_path / "kernels.s"
    src.write_text(KERNELS)
    subprocess.check_call([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", str(src),
                                                         "-o", str(out)])
    writer, seen = {}, 0
    for line in out.read_text().splitlines():
        f = line.split(";")[0].replace(",", " ").split()
        if not f or not f[0].startswith(("v_", "ds_", "global_", "buffer_", "scratch_")):
            continue
        if f[0] == "v_med3_u32":
            seen += 1
            for key in f[3:5]:
                (r,) = _registers(key)
                assert writer.get(r, "").startswith("v_"), (line, writer.get(r))
                assert "mfma" not in writer[r], (line, writer[r])
        for r in _registers(f[1]) if len(f) > 1 else ():
            writer[r] = f[0]
    assert seen >= 4 * 8
