"""Depthwise convolution: operands behind it that depend on the channel alone (loaded once per lane) and ones that depend on
the position, positions of more than 128 vectors (the halo of a tile is then staged in a second round), RELU and NEG on the
packed values with NaN, infinities and signed zeros."""
import pytest

import workloads as wl
from pf_testlib import SPEC_JIT, check_chain, compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


def _chain(dtype, shape, k, stride, pre, operand, seed=0):
    n, h, w, c = shape
    oh, ow = (h - 1) // stride + 1, (w - 1) // stride + 1
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (k, k, c))])
    t = [wl.random_tensor(shape, dtype, 9000 + seed, scale=0.8), wl.random_tensor((k, k, c), dtype, 9001 + seed, scale=1.0 / k)]
    shp = {"channel": (c,), "column": (ow, c), "sample": (n, 1, 1, c), "scalar": (1,), "full": (n, oh, ow, c)}[operand]
    s.inputs.append((dtype, shp))
    t.append(wl.random_tensor(shp, dtype, 9002 + seed, scale=0.5))
    v = 0
    for name in pre:
        v = s.op(name, v)
    v = s.op("dwconv2d", v, 1, i=[stride] if stride != 1 else [])
    s.out(s.op("add", v, 2), dtype)
    return s, t


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("operand", ["channel", "column", "sample", "scalar", "full"])
@pytest.mark.parametrize("k,stride", [(3, 1), (5, 1), (3, 2), (5, 2)])
def test_operands_behind_the_convolution(k, stride, operand, dtype):
    s, t = _chain(dtype, (2, 13, 11, 72), k, stride, ["relu"], operand)
    check_chain(s, t, what=f"{k}x{k}/{stride} + {operand} {dtype}")


@pytest.mark.parametrize("shape,k,dtype", [((1, 9, 3, 1040), 3, "f16"), ((1, 7, 2, 516), 3, "f32"), ((2, 6, 1, 8), 3, "bf16"),
                                           ((1, 7, 5, 1028), 3, "f16")])
def test_wide_positions(shape, k, dtype):
    s, t = _chain(dtype, shape, k, 1, ["relu"], "channel", seed=10)
    check_chain(s, t, what=f"{shape} {k}x{k} {dtype}")


def test_the_widest_5x5_tile():
    # 96 KB of packed LDS tile; the interpreted kernels, whose tile is never packed, do not hold it
    s, t = _chain("f16", (1, 7, 2, 1024), 5, 1, ["relu"], "channel", seed=15)
    outs, info = gpu_run(s, t)
    assert info.spec_id == SPEC_JIT
    compare(outs[0], oracle_run(s, t)[0], "f16", "5x5, 1024 channels")


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_nan_infinities_and_signed_zeros_in_front(dtype):
    for pre in (["relu"], ["neg", "relu"], ["neg"]):
        s, t = _chain(dtype, (1, 12, 12, 16), 3, 1, pre, "channel", seed=20)
        t[0][0, 2, 3, 1], t[0][0, 8, 8, 2], t[0][0, 5, 5, 3] = float("nan"), -float("nan"), -0.0
        t[0][0, 9, 1, 4] = float("inf")      # (RELU of -inf is 0, of +inf an infinity or, beside a zero weight, none)
        check_chain(s, t, what=f"{pre} {dtype}")


@pytest.mark.parametrize("k,stride,dtype,pre", [(3, 1, "f16", "silu"), (3, 2, "f16", "silu"), (5, 2, "bf16", "silu"), (5, 1, "f32", "silu"), (5, 1, "f16", "neg")])
def test_one_kernel_serves_small_and_large_tensors(k, stride, dtype, pre):
    from paper_2307_04995_amd import binding as pf
    s, _ = _chain(dtype, (1, 12, 12, 64), k, stride, [pre, "neg"], "channel", seed=30)
    pf.Plan(s, 0).close()
    compiled = pf.pf_jit_compile_count() + pf.pf_jit_cache_hits()
    s.inputs[0] = (dtype, (64, 112, 112, 64))
    pf.Plan(s, 0).close()
    assert pf.pf_jit_compile_count() + pf.pf_jit_cache_hits() == compiled
