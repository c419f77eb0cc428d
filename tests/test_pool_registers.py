"""The interpreted poolings keep the micro-program's state in registers: the kernels are compiled for the device and their
scratch memory per lane read from the assembly's metadata."""
import os
import re
import subprocess

import pytest

from paper_2307_04995_amd import build


@pytest.mark.skipif(not os.path.exists(build._hipcc()), reason="needs hipcc")
def test_interpreted_kernels_use_no_scratch(tmp_path):
    kernels = [f"pf::pool_kernel<pf::{dt}, {nv}, pf::GenericSpec, {op}, {rg}>"
               for dt, nv, op, rg in (("DT_F16", 8, 2, "false"), ("DT_BF16", 4, 1, "true"), ("DT_F32", 4, 2, "false"))]
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text('#include <hip/hip_runtime.h>\n#include "pf_pool_kernels.hpp"\n' +
                   "".join(f"template __global__ void {k}(const pf::ChainArgs, const pf::PoolGeom);\n" for k in kernels))
    cmd = [build._hipcc()] + build.FLAGS + ["-I" + build.CSRC, "-S", "--cuda-device-only", str(src), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    scratch = [int(v) for v in re.findall(r"\.private_segment_fixed_size: +(\d+)", out.read_text())]
    assert len(scratch) == len(kernels) and max(scratch) == 0, list(zip(scratch, kernels))
