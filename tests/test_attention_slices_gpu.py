"""One-token attention in slices of one to eight steps: caches that end at the edges of a step, heads that are one slice, and the
static call, whose slices are the plan's."""
import pytest
import torch

import workloads as wl
from pf_testlib import check_chain, gpu_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("f16", 64), ("bf16", 128), ("f32", 64), ("f16", 256)])
@pytest.mark.parametrize("steps", [1, 3, 5, 6, 7, 8, 9, 15, 21])
def test_caches_that_end_at_a_step(steps, dtype, d):
    rows = 256 // (d * (4 if dtype == "f32" else 2) // 16)  # of a step
    for t in (rows * steps - 2, rows * steps - 1, rows * steps):
        spec, ins = wl.x2_decode_attention(b=2, h=3, t=t, d=d, dtype=dtype)
        _, info, _ = check_chain(spec, ins, what=f"t={t} d={d} {dtype}")
        if t + 1 <= rows * 8 and steps <= 3:
            assert info.grid[0] == 1


@pytest.mark.parametrize("b,h,t,d", [(1, 3, 100, 64), (2, 5, 700, 64), (4, 32, 600, 128), (8, 32, 1000, 128)])
def test_static_call_takes_the_plans_slices(b, h, t, d):
    from paper_2307_04995_amd import binding as pf
    spec, ins = wl.x2_decode_attention(b=b, h=h, t=t, d=d, dtype="f16")
    planned, _ = gpu_run(spec, ins)
    dev = [x.cuda() for x in ins]
    out = torch.empty_like(dev[0])
    st = pf.pf_chain_run_static(pf.make_desc(spec), 0, [x.data_ptr() for x in dev], [out.data_ptr()], torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    if st == pf.PF_ERR_NOMEM:  # (more partial results than the static scratch array holds)
        assert b * h * ((t + 16) // 64) * 160 * 4 > pf.PF_STATIC_SCRATCH_BYTES // 2
        return
    assert st == pf.PF_OK
    # counted and polled merges weigh the same slices, in other orders where a head has several: fp32 rounding, then fp16's
    assert (out.cpu().float() - planned[0].float()).abs().max() <= 2.0 ** -10 * planned[0].float().abs().max()
