"""GPU parity for GroupNorm over slabs of whole groups (a workgroup owns a slab, or a slice of one): forced onto shapes whose slabs,
steps and slices end everywhere, and where the planner takes it."""
import numpy as np
import pytest
import torch

import workloads as wl
from pf_testlib import check_chain, compare, env, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


def _chain(shape, groups, dtype, act="silu", seed=0, bias=False):
    c = shape[-1]
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (c,)), (dtype, (c,))] + ([(dtype, (c,))] if bias else []))
    v = s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[groups])
    v = s.op(act, v) if act != "none" else v
    s.out(s.op("add", v, 3) if bias else v, dtype)
    t = [wl.random_tensor(shape, dtype, 7300 + seed), wl.random_tensor((c,), dtype, 7301 + seed, dist="positive"), wl.random_tensor((c,), dtype, 7302 + seed, scale=0.5)]
    return s, t + ([wl.random_tensor((c,), dtype, 7303 + seed)] if bias else [])


def _slabs(shape, groups, dtype, slab, slices):
    """(vectors per lane, workgroups, bytes of workspace) of a plan of these slabs and slices; the kernel of whole positions has a
    workspace of 256 bytes at least, and 4, 8, 12 or 16 vectors a lane."""
    vec, samples, positions = (4 if dtype == "f32" else 8), shape[0], int(np.prod(shape[1:-1]))
    per_step = 512 // (slab * (shape[-1] // groups) // vec)
    up = lambda n: (n + 255) // 256 * 256
    blocks = samples * (groups // slab) * slices
    return -(-(-(-positions // slices)) // per_step), -(-blocks // 8) * 8, up(16 * samples * groups * slices) + up(4 * blocks) + 256 if slices > 1 else 0


def _taken(info):
    return info.vectors_per_lane, info.grid[0], info.workspace_bytes


# slab and slices: one position, steps that end inside and at the last position, lanes that are not a divisor of 512, groups inside a
# vector and across two, odd channels to a group, slices that differ by a position and leave the last step empty
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape,groups,slab,slices", [((3, 1, 1, 64), 8, 8, 1), ((2, 8, 8, 64), 8, 2, 1), ((1, 16, 33, 64), 8, 1, 1), ((2, 13, 7, 96), 12, 12, 1),
                                                     ((2, 9, 9, 320), 32, 8, 1), ((1, 20, 20, 160), 32, 32, 1), ((5, 5, 5, 40), 5, 5, 1), ((2, 6, 6, 1184), 32, 32, 1),
                                                     ((9, 7, 7, 128), 32, 8, 1), ((2, 9, 9, 64), 8, 4, 2), ((2, 21, 21, 160), 32, 16, 3), ((1, 12, 11, 64), 4, 4, 5),
                                                     ((3, 33, 31, 96), 12, 12, 7), ((1, 64, 64, 64), 2, 1, 16), ((2, 8, 8, 512), 16, 16, 64), ((1, 56, 56, 128), 8, 4, 30)])
def test_slabs_and_slices(shape, groups, slab, slices, dtype):
    s, t = _chain(shape, groups, dtype)
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS=str(slab), PF_SLAB_SLICES=str(slices)):
        _, info, _ = check_chain(s, t, what=f"groupnorm + silu {shape} / {groups} {dtype}, slabs of {slab} groups, {slices} slices")
    assert info.n_launches == 1


def test_runs_of_slabs():
    # more than 16 vectors a lane, nearly as many workgroups as units: the slices of four slabs of eight are dispatched together
    shape = (10, 53, 60, 512)
    s, t = _chain(shape, 8, "f16", seed=5)
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS="1", PF_SLAB_SLICES="3"):
        _, info, _ = check_chain(s, t, what="groupnorm + silu in runs of four slabs")
    assert _taken(info) == _slabs(shape, 8, "f16", 1, 3) == (17, 240, info.workspace_bytes)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_operands_behind_and_a_large_offset(dtype):
    from paper_2307_04995_amd import binding as pf
    s, t = _chain((2, 10, 10, 96), 12, dtype, act="none", bias=True, seed=10)
    with env(PF_GROUP_SLAB="2"):
        _, info, _ = check_chain(s, t, what="groupnorm + bias in slabs")
    assert info.variant == pf.PF_VARIANT_GROUP_RESIDENT and info.n_launches == 1
    # a common offset of 60 with a spread of 0.5: statistics that cancel would be off by percents
    s, t = _chain((2, 16, 16, 64), 8, dtype, act="none", seed=20)
    t[0] = wl.quantise(wl.widen(wl.random_tensor((2, 16, 16, 64), dtype, 7350, scale=0.5)) + 60.0, dtype)
    for slices in ("1", "4"):
        with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS="4", PF_SLAB_SLICES=slices):
            check_chain(s, t, what=f"groupnorm around an offset, {slices} slices")


@pytest.mark.parametrize("shape,groups,dtype", [((7, 56, 56, 768), 32, "f32"), ((1, 56, 56, 416), 32, "f32"), ((4, 64, 64, 224), 32, "bf16"), ((31, 10, 10, 96), 32, "f16")])
def test_shapes_the_planner_takes_in_slabs(shape, groups, dtype):
    s, t = _chain(shape, groups, dtype, seed=30)
    _, info, _ = check_chain(s, t, what=f"groupnorm + silu {shape} {dtype}")
    assert info.n_launches == 1 and info.lds_bytes != 0


def test_repeated_runs_in_place_and_after_a_wait_that_gave_up():
    from paper_2307_04995_amd import binding as pf
    s, t = _chain((2, 20, 20, 128), 8, "f16", seed=40)
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS="4", PF_SLAB_SLICES="8"):
        plan = pf.Plan(s, 0)
        with env(PF_GROUP_SPIN_LIMIT="1"):
            hasty = pf.Plan(s, 0)
    dev = [x.cuda() for x in t]
    for rep in range(6):  # (both parities of the exchange, more than once)
        x = wl.random_tensor((2, 20, 20, 128), "f16", 7400 + rep)
        dev[0].copy_(x)
        plan.run(dev, [dev[0]])  # in place: a workgroup holds its slice before it stores any of it
        torch.cuda.synchronize()
        compare(dev[0].cpu(), oracle_run(s, [x] + t[1:])[0], "f16", f"run {rep}")
    assert plan.poll_error() == 0
    plan.close()
    # a bounded wait that runs out ends the launch, is reported once, and leaves the plan usable
    out = torch.empty_like(dev[0])
    for _ in range(3):
        hasty.run(dev, [out])
    torch.cuda.synchronize()
    assert hasty.poll_error() in (0, 1) and hasty.poll_error() == 0
    hasty.close()


# the input behind its own normalisation: the value that the kernel holds, for each of its vectors (inputs of a quarter: no result
# reaches 8, from where half a unit of bf16's last place, 2^-5, is more than the bar of 2e-2)
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("behind", ["add", "gate"])
@pytest.mark.parametrize("shape,groups,slab,slices", [((3, 10, 10, 96), 8, 8, 1), ((2, 13, 7, 64), 8, 2, 1), ((2, 21, 21, 160), 32, 16, 3), ((1, 33, 31, 64), 8, 4, 8)])
def test_the_input_behind_its_own_normalisation(shape, groups, slab, slices, behind, dtype):
    c = shape[-1]
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (c,)), (dtype, (c,))])
    v = s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[groups])
    s.out(s.op("add", v, 0) if behind == "add" else s.op("mul", s.op("sigmoid", v), 0), dtype)
    t = [wl.random_tensor(shape, dtype, 7500, scale=0.25), wl.random_tensor((c,), dtype, 7501, dist="positive"), wl.random_tensor((c,), dtype, 7502, scale=0.5)]
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS=str(slab), PF_SLAB_SLICES=str(slices)):
        _, info, _ = check_chain(s, t, what=f"{behind} of x and groupnorm(x) {shape} {dtype}, {slices} slices")
    assert _taken(info) == _slabs(shape, groups, dtype, slab, slices)


@pytest.mark.parametrize("shape,dtype", [((31, 10, 10, 96), "f16"), ((1, 56, 56, 416), "f32"), ((4, 64, 64, 224), "bf16")])
def test_the_input_behind_its_own_normalisation_as_planned(shape, dtype):
    c = shape[-1]
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (c,)), (dtype, (c,))])
    s.out(s.op("add", 0, s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[32])), dtype)
    t = [wl.random_tensor(shape, dtype, 7510, scale=0.25), wl.random_tensor((c,), dtype, 7511, dist="positive"), wl.random_tensor((c,), dtype, 7512, scale=0.5)]
    check_chain(s, t, what=f"x + groupnorm(x) {shape} {dtype}")


# a mask behind the normalisation: the position of each vector
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape,groups,slab,slices", [((3, 10, 40, 96), 8, 8, 1), ((2, 91, 64), 8, 2, 1), ((2, 9, 49, 160), 32, 16, 3), ((1, 33, 31, 64), 8, 4, 8)])
def test_a_mask_behind_the_normalisation(shape, groups, slab, slices, dtype):
    c = shape[-1]
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (c,)), (dtype, (c,))])
    s.out(s.op("causal_mask", s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[groups])), dtype)
    t = [wl.random_tensor(shape, dtype, 7520), wl.random_tensor((c,), dtype, 7521, dist="positive"), wl.random_tensor((c,), dtype, 7522, scale=0.5)]
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS=str(slab), PF_SLAB_SLICES=str(slices)):
        _, info, _ = check_chain(s, t, what=f"causal mask of groupnorm {shape} {dtype}, {slices} slices")
    assert _taken(info) == _slabs(shape, groups, dtype, slab, slices)


def test_a_sample_that_does_not_fit_at_once_stays_two_launches():
    # 400 tiles of 16 steps, but the kernel of these steps needs more registers than it has with 16: 534 tiles of 12 are more than two to a
    # unit, so the call is two launches, which can be recorded
    shape, groups = (1, 160, 160, 512), 32
    s = wl.ChainSpec(inputs=[("f32", shape)] + [("f32", (512,))] * 4)
    v = s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[groups])
    s.out(s.op("gelu_erf", s.op("add", s.op("mul", v, 3), 4)), "f32")
    t = [wl.random_tensor(shape, "f32", 7600)] + [wl.random_tensor((512,), "f32", 7601 + k, dist="positive", scale=0.5) for k in range(4)]
    _, info, _ = check_chain(s, t, what="groupnorm, scale, shift, gelu of a sample of 400 tiles")
    assert info.n_launches == 2


# seven, three and fourteen positions to a lane; a group of equal values is centred to zero exactly, so the result is beta
@pytest.mark.parametrize("shape,groups,slab,slices", [((4, 64, 64, 224), 32, 4, 8), ((1, 56, 56, 416), 32, 4, 26), ((2, 21, 21, 64), 8, 8, 1)])
def test_equal_values_are_their_own_mean(shape, groups, slab, slices):
    c = shape[-1]
    s, t = _chain(shape, groups, "f32", act="none", seed=50)
    level = np.random.default_rng(7700).uniform(500.0, 1000.0, (shape[0], 1, 1, groups, 1)).astype(np.float32)
    t[0] = torch.from_numpy(np.broadcast_to(level, shape[:-1] + (groups, c // groups)).reshape(shape).copy())
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS=str(slab), PF_SLAB_SLICES=str(slices)):
        outs, info = gpu_run(s, t)
    assert _taken(info) == _slabs(shape, groups, "f32", slab, slices)
    assert torch.equal(outs[0], t[2].expand(shape))


@pytest.mark.parametrize("shape,slices", [((4, 64, 64, 224), 8), ((16, 7, 73, 224), 1)])
def test_means_are_not_off_all_the_same_way(shape, slices):
    # Values around 1000, whose last place is 2^-14.  A group's mean is rounded at each level of a tree: 0.41 of that (rms), and the average over
    # 128 groups and more 0.04.  A seventh rounded once for all lanes would put every mean off by 0.7.
    s, t = _chain(shape, 32, "f32", act="none", seed=60)
    t[0], t[1], t[2] = wl.random_tensor(shape, "f32", 7710) + 1000.0, torch.ones(224), torch.zeros(224)
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS="4", PF_SLAB_SLICES=str(slices)):
        outs, info = gpu_run(s, t)
    assert _taken(info) == _slabs(shape, 32, "f32", 4, slices)
    assert abs((outs[0].double().numpy() - oracle_run(s, t)[0]).mean()) <= 0.25 * 2.0 ** -14


@pytest.mark.parametrize("shape,slices", [((8, 32, 14, 512), 1), ((2, 53, 60, 512), 7)])
def test_packed_variances_around_an_offset(shape, slices):
    # Sums of squares around M = 300 with a spread of 1: a rounding of a lane's sum is up to 2^-24 M^2 of the variance, averaged over the lanes of
    # a group.  Half of that for all lanes alike is the bar, a quarter in the scale of the result: 1.3e-3.  Seven positions to a lane, divided by a
    # rounded reciprocal, would be off by 2.3e-3 and more.
    s, t = _chain(shape, 8, "f16", act="none", seed=70)
    t[0] = wl.quantise(wl.widen(wl.random_tensor(shape, "f16", 7720)) + 300.0, "f16")
    t[1], t[2] = torch.ones(512, dtype=torch.float16), torch.zeros(512, dtype=torch.float16)
    with env(PF_GROUP_SLAB="2", PF_SLAB_GROUPS="1", PF_SLAB_SLICES=str(slices)):
        outs, info = gpu_run(s, t)
    assert _taken(info) == _slabs(shape, 8, "f16", 1, slices)
    got, want = outs[0].double().numpy(), oracle_run(s, t)[0]
    assert abs((got * want).sum() / (want * want).sum() - 1.0) <= 300.0 ** 2 * 2.0 ** -26


@pytest.mark.parametrize("shape,dtype,slab,slices", [((31, 10, 10, 96), "f16", 8, 1), ((7, 56, 56, 768), "f32", 8, 9), ((1, 56, 56, 416), "f32", 4, 21), ((4, 64, 64, 224), "bf16", 8, 15)])
def test_the_slabs_that_the_planner_takes(shape, dtype, slab, slices):
    s, t = _chain(shape, 32, dtype, seed=30)
    _, info = gpu_run(s, t)
    assert _taken(info) == _slabs(shape, 32, dtype, slab, slices)
