"""GPU parity for a group normalisation that only a pooling reads: two kernels, neither of which writes the normalised
tensor (the first computes the statistics, the second normalises what it pools)."""
import pytest
import torch

import workloads as wl
from pf_testlib import check_chain, compare, env, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


def _pf():
    from paper_2307_04995_amd import binding as pf
    return pf


def _chain(shape, groups, dtype, pre="none", mid="silu", op="reduce_mean", post="none", seed=0):
    c = shape[-1]
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (c,)), (dtype, (c,))])
    t = [wl.quantise(wl.widen(wl.random_tensor(shape, dtype, 6000 + seed)) + wl.widen(wl.random_tensor((c,), dtype, 6001 + seed, scale=2.0)), dtype),
         wl.random_tensor((c,), dtype, 6002 + seed, dist="positive"), wl.random_tensor((c,), dtype, 6003 + seed, scale=0.3)]
    if pre == "bias":
        s.inputs.append((dtype, (c,)))
        t.append(wl.random_tensor((c,), dtype, 6004 + seed, scale=0.5))
    if pre == "residual":
        s.inputs.append((dtype, shape))
        t.append(wl.random_tensor(shape, dtype, 6005 + seed, scale=0.5))
    if post == "add":
        s.inputs.append((dtype, (shape[0],) + (1,) * (len(shape) - 2) + (c,)))
        t.append(wl.random_tensor(s.inputs[-1][1], dtype, 6006 + seed, scale=0.5))
    v = s.op("add", 0, 3) if pre in ("bias", "residual") else 0
    v = s.op("groupnorm", v, 1, 2, f=[1e-5], i=[groups])
    if mid != "none":
        v = s.op(mid, v)
    v = s.op(op, v, i=list(range(1, len(shape) - 1)))
    if post == "add":
        v = s.op("add", v, len(s.inputs) - 1)
    elif post != "none":
        v = s.op(post, v)
    s.out(v, dtype)
    return s, t


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape,groups", [((2, 12, 12, 64), 8), ((3, 16, 16, 320), 32), ((1, 1, 3, 96), 96), ((5, 40, 31, 48), 3), ((2, 7, 9, 100), 10),
                                          ((2, 5, 5, 1024), 512), ((1, 64, 64, 128), 1)])
def test_shapes(shape, groups, dtype):
    s, t = _chain(shape, groups, dtype)
    _, info, _ = check_chain(s, t, what=f"groupnorm > silu > mean {shape} / {groups} {dtype}")
    assert info.n_kernels == 2 and info.n_launches == 2


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
# positions of more than 512 channels are several channel slabs: groups of 37 and 66 lie across their boundaries, whole vectors and ragged
@pytest.mark.parametrize("shape,groups", [((1, 56, 56, 1184), 32), ((2, 9, 9, 1110), 30), ((3, 14, 5, 1122), 17)])
def test_groups_across_channel_slabs(shape, groups, dtype):
    s, t = _chain(shape, groups, dtype, seed=30)
    with env(PF_NORM_POOL_SLAB="0"):
        _, info, _ = check_chain(s, t, what=f"groupnorm > silu > mean {shape} / {groups} {dtype}")
    assert info.n_launches == 2


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("pre,mid,op,post", [("bias", "none", "reduce_max", "none"), ("residual", "relu", "reduce_mean", "sigmoid"), ("none", "none", "reduce_mean", "add"),
                                             ("residual", "silu", "reduce_max", "add")])
def test_steps_around(pre, mid, op, post, dtype):
    s, t = _chain((3, 20, 9, 72), 9, dtype, pre, mid, op, post, seed=20)
    _, info, _ = check_chain(s, t, what=f"{pre} > groupnorm > {mid} > {op} > {post} {dtype}")
    assert info.n_kernels == 2


def test_a_small_spread_around_a_large_offset():
    # a channel level of 60 with a spread of 0.1 in bf16 (spacing 0.25): statistics that cancel would be off by tens of percent
    shape = (2, 32, 32, 64)
    s, t = _chain(shape, 8, "bf16", mid="none", op="reduce_max")
    t[0] = wl.quantise(wl.widen(wl.random_tensor(shape, "bf16", 6100, scale=0.1)) + 60.0, "bf16")
    outs, _ = gpu_run(s, t)
    with env(PF_NORM_POOL="0"):
        split, info = gpu_run(s, t)
    assert info.n_launches > 2
    want = oracle_run(s, t)[0]
    # (one step of bf16 at the magnitude of the result)
    bar = abs(want).max() * 2.0 ** -7
    assert abs(wl.widen(outs[0]) - want).max() <= bar and abs(wl.widen(split[0]) - want).max() <= bar


def test_repeated_runs_and_replays_of_a_graph():
    pf = _pf()
    s, t = _chain((4, 24, 24, 320), 32, "f16")
    plan = pf.Plan(s, 0)
    dev = [x.cuda() for x in t]
    out = torch.empty(plan.output_shapes()[0], dtype=torch.float16, device="cuda")
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        plan.run(dev, [out])
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            plan.run_ptrs([x.data_ptr() for x in dev], [out.data_ptr()], torch.cuda.current_stream().cuda_stream)
    for rep in range(4):
        x = wl.random_tensor((4, 24, 24, 320), "f16", 6200 + rep)
        dev[0].copy_(x)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        compare(out.cpu(), oracle_run(s, [x] + t[1:])[0], "f16", f"replay {rep}")
        plan.run(dev, [out])
        torch.cuda.synchronize()
        compare(out.cpu(), oracle_run(s, [x] + t[1:])[0], "f16", f"eager run {rep}")
    assert plan.poll_error() == 0
    plan.close()


@pytest.mark.parametrize("mid", ["tanh", "sigmoid", "silu", "gelu_erf", "exp"])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_steps_in_between_are_as_exact_as_in_fp32(dtype, mid):
    # Between normalisation and pooling the values are fp32 and no tensor of 16 bits: near zero, where tanh by way of 2 sigmoid(2 x)
    # - 1 keeps 1e-7 of 1, and with the result scaled up so that its rounding to the storage type (half a step, 2^-11 or 2^-8 of
    # the value) is all the error there is, beside 1e-5 for the fp32 steps and, for GELU, the 3e-7 |x| of its approximation.
    s, t = _chain((2, 12, 12, 64), 8, dtype, mid="none")
    t[1] = torch.full((64,), 2.0 ** -15 if mid in ("tanh", "gelu_erf", "silu") else 1.0).to(t[1].dtype)
    t[2] = torch.zeros_like(t[2])
    s = wl.ChainSpec(inputs=s.inputs)
    v = s.op(mid, s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[8]))
    v = s.op("reduce_max", v, i=[1, 2])
    s.out(s.op("scale", v, f=[2.0 ** 14]), dtype) if mid in ("tanh", "gelu_erf", "silu") else s.out(v, dtype)
    outs, info = gpu_run(s, t)
    assert info.n_launches == 2
    want = oracle_run(s, t)[0]
    got = wl.widen(outs[0])
    bar = (2.0 ** -11 if dtype == "f16" else 2.0 ** -8) + 1e-5
    assert (abs(got - want) / abs(want)).max() <= bar
    # ... and against the chain as kernels of its own on fp32 copies: the same value, or the next one where it lies halfway
    with env(PF_NORM_POOL="0"):
        split, info = gpu_run(s, t)
    assert info.n_launches > 2
    assert (abs(got - wl.widen(split[0])) / abs(want)).max() <= 2.0 * bar
    assert (got != wl.widen(split[0])).mean() < 0.02


@pytest.mark.parametrize("mid", ["sigmoid", "silu", "tanh"])
def test_infinities_and_nan_in_between(mid):
    # a residual of +-inf, NaN and the lowest value joins behind the normalisation
    shape = (1, 4, 4, 64)
    s, t = _chain(shape, 8, "f16", mid="none", seed=40)
    y = wl.random_tensor(shape, "f16", 6300)
    y[0, 1, 1, 3], y[0, 2, 2, 9], y[0, 0, 3, 17], y[0, 3, 0, 33], y[0, 3, 1, 40] = float("inf"), -float("inf"), float("nan"), 9.0, -65504.0
    s = wl.ChainSpec(inputs=s.inputs + [("f16", shape)])
    v = s.op("add", s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[8]), 3)
    s.out(s.op("reduce_sum", s.op(mid, v), i=[1, 2]), "f16")
    outs, info = gpu_run(s, t + [y])
    assert info.n_launches == 2
    compare(outs[0], oracle_run(s, t + [y])[0], "f16", f"infinities in front of {mid}")
