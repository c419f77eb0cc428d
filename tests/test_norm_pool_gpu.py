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
