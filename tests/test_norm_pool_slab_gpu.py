"""GPU parity for GroupNorm, the steps behind it and a pooling in one launch: a workgroup holds a slab of whole groups."""
import pytest
import torch

import workloads as wl
from pf_testlib import check_chain, compare, env, gpu_run, oracle_run
from test_norm_pool_gpu import _chain

pytestmark = pytest.mark.gpu


# groups inside, across and at the edges of 16-byte vectors; positions fewer than, equal to and one more than whole steps
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape,groups", [((2, 12, 12, 64), 8), ((3, 16, 16, 320), 32), ((1, 1, 3, 96), 96), ((5, 40, 31, 48), 3), ((1, 13, 79, 40), 4),
                                          ((2, 5, 5, 1024), 512), ((2, 1, 511, 24), 8), ((2, 1, 513, 24), 8), ((1, 2, 256, 1184), 32), ((2, 3, 1, 8), 1)])
def test_shapes(shape, groups, dtype):
    s, t = _chain(shape, groups, dtype, seed=60)
    with env(PF_NORM_POOL_SLAB="2"):
        _, info, _ = check_chain(s, t, what=f"one launch: groupnorm > silu > mean {shape} / {groups} {dtype}")
    assert info.n_kernels == 1 and info.n_launches == 1 and info.workspace_bytes == 0


@pytest.mark.parametrize("dtype", ["f16", "f32"])
# (no sum of 180 values: above 32 half a step of fp16, 2^-11 of the value, is past the absolute bar of 2e-2)
@pytest.mark.parametrize("mid,op,post", [("none", "reduce_max", "none"), ("relu", "reduce_mean", "sigmoid"), ("silu", "reduce_mean", "add")])
def test_steps_around(mid, op, post, dtype):
    s, t = _chain((3, 20, 9, 72), 9, dtype, "none", mid, op, post, seed=70)
    with env(PF_NORM_POOL_SLAB="2"):
        _, info, _ = check_chain(s, t, what=f"one launch: groupnorm > {mid} > {op} > {post} {dtype}")
    assert info.n_kernels == 1


def test_operands_read_at_every_position_take_two_launches():
    s, t = _chain((2, 12, 12, 64), 8, "f16", pre="bias", seed=80)
    with env(PF_NORM_POOL_SLAB="2"):
        _, info, _ = check_chain(s, t, what="bias > groupnorm > silu > mean")
    assert info.n_kernels == 2


def test_taken_by_size():
    s, t = _chain((31, 16, 16, 1152), 32, "bf16", seed=90)
    _, info, _ = check_chain(s, t, what="one launch by the rule")
    assert info.n_launches == 1


def test_a_small_spread_around_a_large_offset():
    # a channel level of 60 with a spread of 0.1 in bf16 (spacing 0.25): statistics that cancel would be off by tens of percent
    shape = (2, 32, 32, 64)
    s, t = _chain(shape, 8, "bf16", mid="none", op="reduce_max")
    t[0] = wl.quantise(wl.widen(wl.random_tensor(shape, "bf16", 6100, scale=0.1)) + 60.0, "bf16")
    with env(PF_NORM_POOL_SLAB="2"):
        outs, info = gpu_run(s, t)
    assert info.n_launches == 1
    want = oracle_run(s, t)[0]
    # (one step of bf16 at the magnitude of the result)
    assert abs(wl.widen(outs[0]) - want).max() <= abs(want).max() * 2.0 ** -7


@pytest.mark.parametrize("mid,op", [("silu", "reduce_max"), ("none", "reduce_mean")])
def test_an_infinity_or_nan_stays_in_its_group(mid, op):
    # groups of ten channels: neighbours share a vector
    shape = (2, 12, 12, 40)
    s, t = _chain(shape, 4, "f16", mid=mid, op=op, seed=95)
    t[0][0, 3, 4, 13], t[0][0, 11, 11, 39], t[0][1, 0, 0, 20] = float("inf"), -float("inf"), float("nan")
    with env(PF_NORM_POOL_SLAB="2"):
        outs, info = gpu_run(s, t)
    assert info.n_launches == 1
    want = oracle_run(s, t)[0]
    assert wl.widen(outs[0]).size == 80 and torch.isnan(outs[0]).sum() == 30
    compare(outs[0], want, "f16", f"infinities and NaN in front of groupnorm > {mid} > {op}")


def test_repeated_runs_and_replays_of_a_graph():
    from paper_2307_04995_amd import binding as pf
    shape = (31, 16, 16, 1152)
    s, t = _chain(shape, 32, "f16", seed=97)
    plan = pf.Plan(s, 0)
    assert plan.info().n_launches == 1
    dev = [x.cuda() for x in t]
    out = torch.empty(plan.output_shapes()[0], dtype=torch.float16, device="cuda")
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        plan.run(dev, [out])
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            plan.run_ptrs([x.data_ptr() for x in dev], [out.data_ptr()], torch.cuda.current_stream().cuda_stream)
    for rep in range(3):
        x = wl.random_tensor(shape, "f16", 6400 + rep)
        want = oracle_run(s, [x] + t[1:])[0]
        dev[0].copy_(x)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        compare(out.cpu(), want, "f16", f"replay {rep}")
        out.zero_()
        plan.run(dev, [out])
        torch.cuda.synchronize()
        compare(out.cpu(), want, "f16", f"eager run {rep}")
    plan.close()


@pytest.mark.parametrize("shape,dtype", [((32, 64, 64, 320), "f16"), ((19, 14, 14, 576), "bf16"), ((21, 28, 28, 64), "f16"), ((23, 32, 32, 992), "bf16"), ((8, 56, 56, 256), "bf16")])
def test_shapes_of_more_than_two_mebibytes(shape, dtype):
    s, t = _chain(shape, 32, dtype, seed=91)
    _, info, _ = check_chain(s, t, what=f"groupnorm > silu > mean {shape} {dtype}, as planned")
    assert info.n_kernels == 1 and info.workspace_bytes == 0


# 28, 14 and 7 positions to a lane: a group of equal values is centred to zero exactly, so its pooled value is beta
@pytest.mark.parametrize("shape,groups", [((8, 28, 64, 64), 1), ((8, 28, 32, 128), 2), ((8, 7, 64, 64), 1)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_equal_values_are_their_own_mean(shape, groups, dtype):
    s, t = _chain(shape, groups, dtype, mid="none", seed=98)
    level = wl.random_tensor((shape[0], 1, 1, groups, 1), dtype, 6500, dist="uniform", scale=250.0) + 750.0
    t[0] = level.expand(shape[:-1] + (groups, shape[-1] // groups)).reshape(shape).contiguous()
    with env(PF_NORM_POOL_SLAB="2"):
        outs, info = gpu_run(s, t)
    assert info.n_launches == 1
    assert torch.equal(outs[0].reshape(shape[0], -1), t[2].expand(shape[0], -1))
