"""The column family's workgroup sizes: 256, 512 or 1024 lanes share a slab, chosen by how many slabs there are.  Column
lengths around the steps of every size, with slab counts that are no multiple of the eight compute dies."""
import pytest
import torch

import workloads as wl
from pf_testlib import check_chain, env, gpu_run

pytestmark = pytest.mark.gpu


def _chain(dtype, shape, kind="layernorm"):
    n, c = shape[0], shape[1]
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (c,))] + ([(dtype, (c,))] if kind == "layernorm" else []))
    v = s.op("permute", 0, i=[0, 2, 3, 1])
    v = s.op("layernorm", v, 1, 2, f=[1e-6]) if kind == "layernorm" else s.op("rmsnorm", v, 1, f=[1e-6])
    s.out(s.op("permute", v, i=[0, 3, 1, 2]), dtype)
    t = [wl.random_tensor(shape, dtype, 7700 + c), wl.random_tensor((c,), dtype, 7701, dist="positive")]
    return s, t + ([wl.random_tensor((c,), dtype, 7702, scale=0.3)] if kind == "layernorm" else [])


@pytest.mark.parametrize("threads", [256, 512, 1024])
@pytest.mark.parametrize("shape,dtype", [((3, 2, 4, 4), "f16"), ((11, 130, 7, 7), "f16"), ((1, 192, 14, 14), "bf16"), ((3, 256, 9, 9), "f32"), ((2, 257, 14, 14), "f16"),
                                         ((5, 384, 5, 9), "bf16"), ((1, 640, 8, 8), "f32"), ((1, 769, 7, 7), "f16"), ((1, 1023, 6, 6), "f32"), ((1, 1024, 14, 14), "f16")])
def test_every_size(shape, dtype, threads):
    if threads == 512 and shape[1] > 256:
        pytest.skip("512 lanes are built for columns of at most 256")
    for kind in ("layernorm", "rmsnorm"):
        s, t = _chain(dtype, shape, kind)
        with env(PF_COL_THREADS=threads):
            _, info, _ = check_chain(s, t, what=f"{kind} {shape} {dtype} on {threads} lanes")
        assert info.block[0] == threads


def test_sizes_agree_and_the_planner_chooses():
    s, t = _chain("f32", (40, 300, 12, 12))   # 200 slabs
    few, info = gpu_run(s, t)
    assert info.block[0] == 1024
    with env(PF_COL_THREADS=256):
        small, _ = gpu_run(s, t)
    assert (few[0] - small[0]).abs().max() < 2e-6   # sums of 300 values in another order, results of magnitude 4
    s, t = _chain("f16", (70, 40, 24, 24))    # 700 slabs of short columns
    _, info, _ = check_chain(s, t, what="many slabs")
    assert info.block[0] == 256
