"""A pooling's position rows are merged by as many lanes to a channel as fit the workgroup: channel counts at the steps of that
number (64 lanes down to one), one slice to a slab and several, positions fewer than the lanes."""
import pytest

import workloads as wl
from pf_testlib import check_chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["reduce_mean", "reduce_max"])
@pytest.mark.parametrize("dtype,channels", [("f16", c) for c in (3, 8, 9, 16, 24, 40, 64, 72, 128, 136, 256, 264, 512)] + [("f32", 4), ("f32", 12), ("f32", 260)])
def test_lanes_to_a_channel(dtype, channels, op):
    for positions in (1, 3, 70, 5000):
        shape = (2, positions, channels)
        s = wl.ChainSpec(inputs=[(dtype, shape)])
        s.out(s.op(op, 0, i=[1]), dtype)
        check_chain(s, [wl.random_tensor(shape, dtype, 7000 + channels)], what=f"{op} {shape} {dtype}")
