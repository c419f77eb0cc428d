"""The staged convolution keeps what it works on in registers, whatever stands in front of it: its kernels are compiled for the
device and their scratch memory per lane (spilled registers) read from the assembly's metadata."""
import os
import re
import subprocess

import pytest

from paper_2307_04995_amd import build

# micro-op codes and operand kinds of pf_common.h
MOV, ADD, RELU, SILU = 0, 1, 10, 12
FULL, VEC = 2, 3


def _step(code, kind=0, slot=0):
    return code | (kind << 8) | (slot << 16)


PROLOGUES = {
    "relu": [_step(MOV, FULL, 0), _step(RELU)],
    "silu": [_step(MOV, FULL, 0), _step(SILU)],
    "bias > relu": [_step(MOV, FULL, 0), _step(ADD, VEC, 0), _step(RELU)],
    "residual > silu": [_step(MOV, FULL, 0), _step(ADD, FULL, 1), _step(SILU)],
    "three operands": [_step(MOV, FULL, 0), _step(ADD, FULL, 1), _step(ADD, FULL, 2)],
}


def _kernel(dtype, prologue, ragged):
    """The template-id of the 3 x 3 kernel with a bias behind it; slots: the prologue's vectors, the kernels, the bias."""
    n_full = sum((u >> 8 & 255) == FULL for u in prologue)
    n_vec = sum((u >> 8 & 255) == VEC for u in prologue)
    steps = ", ".join(f"{u}u" for u in prologue)
    spec = f"pf::StaticSpec<{n_full}, {n_vec + 2}, 0, pf::CORE_DWCONV, {n_vec}, -1, pf::StaticList<{steps}>, pf::StaticList<{_step(ADD, VEC, n_vec + 1)}u>, 4>"
    return f"pf::dwconv_staged_kernel<{dtype}, {spec}, 3, {ragged}>"


@pytest.mark.skipif(not os.path.exists(build._hipcc()), reason="needs hipcc")
def test_staged_kernels_do_not_spill(tmp_path):
    kernels = [_kernel(f"pf::{dt}", p, rg) for dt in ("DT_F32", "DT_F16", "DT_BF16") for p in PROLOGUES.values() for rg in ("false", "true")]
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text('#include <hip/hip_runtime.h>\n#include "pf_stencil_kernels.hpp"\n' +
                   "".join(f"template __global__ void {k}(const pf::ChainArgs, const pf::StencilGeom);\n" for k in kernels))
    cmd = [build._hipcc()] + build.FLAGS + ["-I" + build.CSRC, "-S", "--cuda-device-only", str(src), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    scratch = [int(v) for v in re.findall(r"\.private_segment_fixed_size: +(\d+)", out.read_text())]
    assert len(scratch) == len(kernels) and max(scratch) == 0, list(zip(scratch, kernels))
