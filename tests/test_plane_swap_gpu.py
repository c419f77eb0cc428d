"""Layout-only swaps of a plane's two dimensions with an extent that is not a whole number of 16-byte vectors: bit-exact on
arbitrary bits, strips that are one stretch of the input or of the output, partial first, last and only vectors."""
import numpy as np
import pytest
import torch

import workloads as wl
from pf_testlib import env

pytestmark = pytest.mark.gpu


def _run(shape, perm, dtype, planes, seed, **flags):
    from paper_2307_04995_amd import binding as pf
    g = np.random.default_rng(seed)
    udt, tdt = (np.int32, torch.float32) if dtype == "f32" else (np.int16, torch.float16 if dtype == "f16" else torch.bfloat16)
    info_t = np.iinfo(udt)
    bits = g.integers(info_t.min, info_t.max, shape, dtype=udt, endpoint=True)
    s = wl.ChainSpec(inputs=[(dtype, tuple(shape))])
    s.out(s.op("permute", 0, i=perm), dtype)
    x = torch.from_numpy(bits).cuda().view(tdt)
    pad = 64
    n = bits.size
    buf = torch.full((n + 2 * pad,), 7, dtype=torch.int32 if dtype == "f32" else torch.int16, device="cuda")
    with env(**flags):
        plan = pf.Plan(s, 0)
    plan.run_ptrs([x.data_ptr()], [buf[pad:].data_ptr()], torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert (got[:pad] == 7).all() and (got[pad + n:] == 7).all(), "wrote outside the output"
    assert np.array_equal(got[pad:pad + n].reshape(bits.transpose(perm).shape), bits.transpose(perm)), (shape, perm, dtype)
    grid = plan.info().grid[0]
    plan.close()
    return grid


# the strip is 64 16-bit or 32 fp32 rows (half of that for rows of more than about 500 elements): extents on both sides of
# it, flat inputs (input rows not whole vectors) and flat outputs (output rows not whole vectors), rows up to the longest
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("a,b", [(2, 3), (64, 7), (65, 49), (384, 196), (63, 197), (100, 64), (33, 72), (7, 8), (129, 500), (40, 1001), (1001, 40), (500, 24), (13, 1021),
                                 (2, 1030)])
def test_planes(a, b, dtype):
    for planes in (1, 3) if a * b > 6000 else (1, 3, 300):
        _run((planes, a, b), [0, 2, 1], dtype, planes, 8000 + a)


def test_feature_maps_and_what_stays_on_tiles():
    # [n, c, h, w] <-> [n, h, w, c] with 14 x 14 positions, 19 planes: strips are not a multiple of the dies
    strips = _run((19, 72, 14, 14), [0, 2, 3, 1], "f16", 19, 8101)
    assert strips == (19 * 2 + 7) // 8 * 8
    # (a flat output takes 512 strips at least: 260 planes of two)
    assert _run((260, 14, 14, 72), [0, 3, 1, 2], "f16", 260, 8102) == (260 * 2 + 7) // 8 * 8
    _run((19, 14, 14, 72), [0, 3, 1, 2], "f16", 19, 8106)
    for shape in ((520, 33, 16), (260, 3, 72), (172, 101, 136), (520, 900, 24)):   # flat outputs: a last strip that is not full, a partial step of the walk
        for dtype in ("f16", "f32"):
            _run(shape, [0, 2, 1], dtype, shape[0], 8107)
    _run((3, 1500, 1201), [0, 2, 1], "f16", 3, 8103)     # rows too long for a strip in LDS
    _run((5, 6, 7, 9), [3, 1, 2, 0], "f32", 1, 8104)     # not a swap of adjacent dimensions
    _run((4, 3, 50, 11), [1, 0, 3, 2], "bf16", 1, 8105)  # the planes change places as well


def test_more_planes_than_a_launch_has_strips():
    from paper_2307_04995_amd import binding as pf
    planes = (1 << 24) + 5000
    s = wl.ChainSpec(inputs=[("f16", (planes, 3, 5))])
    s.out(s.op("permute", 0, i=[0, 2, 1]), "f16")
    x = torch.randint(-30000, 30000, (planes, 3, 5), dtype=torch.int16, device="cuda")
    out = torch.zeros((planes, 5, 3), dtype=torch.int16, device="cuda")
    plan = pf.Plan(s, 0)
    plan.run([x.view(torch.float16)], [out.view(torch.float16)])
    assert torch.equal(out, x.transpose(1, 2))
    plan.close()
