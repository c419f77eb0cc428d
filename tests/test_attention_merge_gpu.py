"""The merge of a head's slices reads one, two or eight slices per thread group at a time (256 / d groups): slice counts on
both sides of each step and of a whole round, repeated launches on one plan (the words are put back after every launch)."""
import pytest
import torch

import workloads as wl
from pf_testlib import check_chain, compare, env, oracle_run

pytestmark = pytest.mark.gpu


# 4 steps of 256 / (d / 8) rows per slice with 16-bit types: 128 rows for d = 64 (4 groups), 64 for d = 128 (2), 32 for d = 256 (1)
@pytest.mark.parametrize("dtype,d,rows", [("f16", 64, 128), ("bf16", 128, 64), ("f16", 256, 32), ("f32", 32, 128), ("f32", 64, 64)])
@pytest.mark.parametrize("splits", [1, 2, 3, 4, 5, 8, 9, 17, 33, 40])
def test_slice_counts(splits, dtype, d, rows):
    spec, ins = wl.x2_decode_attention(b=1, h=3, t=rows * (splits - 1) + 4, d=d, dtype=dtype, salt=splits)
    with env(PF_ATTN_NV="4"):
        _, info, _ = check_chain(spec, ins, what=f"attention d={d} {dtype} in {splits} slices")
    assert info.grid[0] == splits


def test_repeated_launches_and_a_peaked_head():
    from paper_2307_04995_amd import binding as pf
    spec, ins = wl.x2_decode_attention(b=2, h=4, t=3000, d=64, dtype="f16", salt=77)
    plan = pf.Plan(spec, 0)
    out = torch.empty((2, 4, 64), dtype=torch.float16, device="cuda")
    for rep in range(4):
        ins[0] = wl.random_tensor((2, 4, 64), "f16", 9300 + rep, scale=1.0 + 4.0 * rep)   # ever more peaked scores
        dev = [t.cuda() for t in ins]
        plan.run(dev, [out])
        torch.cuda.synchronize()
        compare(out.cpu(), oracle_run(spec, ins)[0], "f16", f"launch {rep}")
    assert plan.poll_error() == 0
    plan.close()
