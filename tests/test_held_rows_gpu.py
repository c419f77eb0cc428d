"""GPU parity for long rows held packed in one workgroup's registers: vectors on a grid of memory lines, so a row's first
and last vectors are partial or absent at every place a row can start within a line."""
import numpy as np
import pytest
import torch

import workloads as wl
from pf_testlib import check_chain, gpu_run, oracle_run

pytestmark = pytest.mark.gpu


def _pf():
    from paper_2307_04995_amd import binding as pf
    return pf


def _softmax(rows, n, dtype, scale=None):
    s = wl.ChainSpec(inputs=[(dtype, (rows, n))])
    v = s.op("scale", 0, f=[scale]) if scale else 0
    s.out(s.op("softmax", v), dtype)
    return s, [wl.random_tensor((rows, n), dtype, 5000 + n % 89, scale=3.0)]


# 36 793 / 36 794 16-bit elements: the last row length of nine vectors a lane and the first of ten; 163 769 the longest row
@pytest.mark.parametrize("n,dtype", [(32769, "f16"), (32776, "bf16"), (36793, "bf16"), (36794, "f16"), (50257, "bf16"), (50264, "f16"), (131071, "f16"),
                                     (163769, "bf16"), (16388, "f32"), (50257, "f32"), (81884, "f32")])
def test_long_softmax(n, dtype):
    rows = 67 if n < 40000 else 11   # odd lengths: every place within a 128-byte line
    spec, ins = _softmax(rows, n, dtype, scale=0.5)
    _, info, _ = check_chain(spec, ins, what=f"held softmax {n} {dtype}")
    assert info.block[0] * info.vectors_per_lane * 16 >= n * ins[0].element_size()


@pytest.mark.parametrize("rows,n,dtype", [(520, 4097, "f16"), (513, 20001, "bf16"), (515, 2051, "f32"), (512, 16381, "f32")])
def test_ragged_softmax_of_many_rows(rows, n, dtype):
    spec, ins = _softmax(rows, n, dtype)
    _, info, _ = check_chain(spec, ins, what=f"held ragged softmax {rows} {n} {dtype}")
    assert info.block[0] * info.vectors_per_lane * 16 >= n * ins[0].element_size()


@pytest.mark.parametrize("n,dtype", [(33001, "f16"), (33008, "bf16"), (20003, "f32")])
def test_normalisations_with_parameters_and_a_second_output(n, dtype):
    rows = 9
    x = wl.random_tensor((rows, n), dtype, 5101, scale=0.6)
    bias, beta = wl.random_tensor((n,), dtype, 5102, scale=0.4), wl.random_tensor((n,), dtype, 5104, scale=0.3)
    gamma = wl.random_tensor((n,), dtype, 5103, dist="positive")
    s = wl.ChainSpec(inputs=[(dtype, (rows, n))] + [(dtype, (n,))] * 3)
    h = s.op("add", 0, 1)
    s.out(s.op("gelu_erf", s.op("layernorm", h, 2, 3, f=[1e-5])), dtype)
    s.out(h, dtype)
    check_chain(s, [x, bias, gamma, beta], what=f"held layernorm {n} {dtype}")
    s = wl.ChainSpec(inputs=[(dtype, (rows, n)), (dtype, (n,))])
    s.out(s.op("rmsnorm", s.op("relu", 0), 1, f=[1e-6]), dtype)
    check_chain(s, [x, gamma], what=f"held rmsnorm {n} {dtype}")


@pytest.mark.parametrize("op", ["reduce_sum", "reduce_max", "reduce_mean"])
@pytest.mark.parametrize("n,dtype", [(40003, "f16"), (17001, "f32")])
def test_reductions(op, n, dtype):
    # all values below zero, shifted: neither a padding zero nor a neighbouring row's value may enter
    x = wl.quantise(-np.abs(wl.widen(wl.random_tensor((7, n), dtype, 5201))).astype(np.float32) - 0.5, dtype)
    s = wl.ChainSpec(inputs=[(dtype, (7, n))])
    v = s.op("scale", 0, f=[0.125 / n if op == "reduce_sum" else 0.5])
    s.out(s.op("scale", s.op(op, v), f=[0.5]), dtype)
    check_chain(s, [x], what=f"held {op} {n} {dtype}")


def test_infinities_and_nan():
    n = 50257
    x = wl.random_tensor((6, n), "f16", 5301, scale=2.0)
    x[0, 0] = float("-inf")
    x[1, :] = float("-inf")          # a row of nothing but -inf is NaN by definition
    x[2, n - 1] = float("nan")
    x[3, 17] = float("inf")
    x[4, :] = 65504.0                # the largest values: the common maximum is far from zero
    s = wl.ChainSpec(inputs=[("f16", (6, n))])
    s.out(s.op("softmax", 0), "f16")
    check_chain(s, [x], what="held softmax, infinities and NaN")


def test_large_common_offset_and_in_place():
    # normalised over a spread of 0.5 around 300 in fp32 (spacing 3e-5): held to 1e-4; the output may be the input
    rows, n = 3, 40001
    x = wl.random_tensor((rows, n), "f32", 5401, scale=0.5) + 300.0
    gamma, beta = wl.random_tensor((n,), "f32", 5402, dist="positive"), wl.random_tensor((n,), "f32", 5403, scale=0.5)
    s = wl.ChainSpec(inputs=[("f32", (rows, n)), ("f32", (n,)), ("f32", (n,))])
    s.out(s.op("layernorm", 0, 1, 2, f=[1e-5]), "f32")
    outs, _ = gpu_run(s, [x, gamma, beta])
    want = oracle_run(s, [x, gamma, beta])[0]
    assert np.abs(wl.widen(outs[0]) - want).max() < 1e-4
    pf = _pf()
    plan = pf.Plan(s, 0)
    buf, gd, bd = x.cuda(), gamma.cuda(), beta.cuda()
    plan.run([buf, gd, bd], [buf])
    torch.cuda.synchronize()
    assert torch.equal(buf.cpu(), outs[0])


@pytest.mark.parametrize("rows,n", [(4, 50257), (4, 50264), (520, 4097)])
@pytest.mark.parametrize("value", [-1e10, 1e10, float(torch.finfo(torch.bfloat16).min), float(torch.finfo(torch.bfloat16).max)])
def test_rows_masked_throughout(value, rows, n):
    # a row of one large value (everything masked with -1e10 or the type's lowest value) is 1 / n per element: the exponent is
    # zero whatever the maximum's product with log2 e rounds to
    for scale in (None, 0.5):
        s, t = _softmax(rows, n, "bf16", scale)
        t[0][0, :], t[0][rows - 1, :] = value, value
        t[0][1, n // 2:] = value
        outs, info, _ = check_chain(s, t, what=f"bf16 softmax of rows of {value}, scale {scale}")
        assert info.block[0] * info.vectors_per_lane * 16 >= n * 2
        for r in (0, rows - 1):
            assert torch.equal(outs[0][r], torch.full((n,), 1.0 / n).to(torch.bfloat16))
    # the same from a mask that is added in front, to rows of one value each (what fp32 makes of -1e10 + logits is another matter)
    s = wl.ChainSpec(inputs=[("bf16", (rows, n)), ("bf16", (n,))])
    s.out(s.op("softmax", s.op("add", 0, 1)), "bf16")
    x = (torch.arange(rows).reshape(rows, 1) % 3).expand(rows, n).to(torch.bfloat16).contiguous()
    outs, _, _ = check_chain(s, [x, torch.full((n,), value, dtype=torch.bfloat16)], what=f"bf16 softmax behind a mask of {value}")
    assert torch.equal(outs[0], torch.full((rows, n), 1.0 / n).to(torch.bfloat16))


@pytest.mark.parametrize("scale", [None, 10.0, 12.0, 1e5])
def test_the_largest_fp16_scores(scale):
    # 65504 times the scale, on both sides of 2^20 (a scale of 11.1); neighbours of the maximum and a second value far below it
    rows, n = 3, 50257
    s, t = _softmax(rows, n, "f16", scale)
    t[0][:] = -65504.0
    t[0][0, :] = 65504.0
    t[0][1, n - 40000:] = 65504.0
    t[0][2, 5::7] = 65472.0
    outs, _, _ = check_chain(s, t, what=f"fp16 softmax of the largest values, scale {scale}")
    for row, count in ((0, n), (1, 40000), (2, len(range(5, n, 7)))):
        assert torch.equal(outs[0][row], torch.where(t[0][row] > 0, 1.0 / count, 0.0).to(torch.float16))


@pytest.mark.parametrize("n", [33001, 33000])
def test_a_causal_mask_that_stays_a_step(n):
    # the value in front of the mask is an output too, so the mask is a step of its own and nothing is skipped: columns are counted
    # from the row's first element, which lies inside the first vector
    s = wl.ChainSpec(inputs=[("bf16", (5, n))])
    h = s.op("scale", 0, f=[0.5])
    s.out(s.op("softmax", s.op("causal_mask", h)), "bf16")
    s.out(h, "bf16")
    _, info, _ = check_chain(s, [wl.random_tensor((5, n), "bf16", 5601, scale=2.0)], what=f"masked softmax and what is in front of it, n {n}")
    assert info.block[0] * info.vectors_per_lane * 16 >= n * 2
