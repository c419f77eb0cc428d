"""GPU parity for the one-launch GroupNorm whose workgroups own whole positions, on shapes that slabs of whole groups take by default."""
import pytest

import workloads as wl
from pf_testlib import check_chain, env

pytestmark = pytest.mark.gpu


# groups of whole vectors, of parts of one and across two; one position, tiles that end inside and at the last one
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("behind", ["silu", "add", "gate", "mask"])
@pytest.mark.parametrize("shape,groups", [((3, 1, 1, 64), 8), ((2, 8, 8, 512), 16), ((2, 13, 7, 96), 12), ((1, 20, 20, 160), 32), ((5, 5, 5, 40), 5)])
def test_steps_behind_whole_positions(shape, groups, behind, dtype):
    c = shape[-1]
    s = wl.ChainSpec(inputs=[(dtype, shape), (dtype, (c,)), (dtype, (c,))])
    v = s.op("groupnorm", 0, 1, 2, f=[1e-5], i=[groups])
    s.out({"silu": lambda: s.op("silu", v), "add": lambda: s.op("add", v, 0), "gate": lambda: s.op("mul", s.op("sigmoid", v), 0), "mask": lambda: s.op("causal_mask", v)}[behind](), dtype)
    # (inputs of a quarter: no result reaches 8, from where half a unit of bf16's last place is more than the bar of 2e-2)
    t = [wl.random_tensor(shape, dtype, 7800, scale=0.25), wl.random_tensor((c,), dtype, 7801, dist="positive"), wl.random_tensor((c,), dtype, 7802, scale=0.5)]
    with env(PF_GROUP_SLAB="0"):
        _, info, _ = check_chain(s, t, what=f"{behind} behind groupnorm over whole positions {shape} {dtype}")
    assert info.n_launches == 1 and info.workspace_bytes >= 256  # (slabs of one slice have none)
