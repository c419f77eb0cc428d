"""Rows on fewer lanes with three or more vectors each: row lengths at the edges of every choice, whole and ragged, causal and not."""
import pytest

import workloads as wl
from pf_testlib import check_chain

pytestmark = pytest.mark.gpu


def _softmax(dtype, rows, n, causal, what):
    s = wl.ChainSpec(inputs=[(dtype, (rows // 64, 64, n))])
    v = s.op("scale", 0, f=[0.125])
    s.out(s.op("softmax", s.op("causal_mask", v) if causal else v), dtype)
    return check_chain(s, [wl.random_tensor((rows // 64, 64, n), dtype, 7500 + n % 89, scale=2.0)], what=what)


# vectors of a row: 33, 41, 48 | 49 (not) | 65, 80 | 81 (not) | 129, 192 | 193 (not), on 16, 32 and 64 lanes
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("vectors,lanes", [(33, 16), (41, 16), (48, 16), (49, 0), (65, 32), (80, 32), (81, 0), (129, 64), (192, 64), (193, 0)])
@pytest.mark.parametrize("dtype,ragged", [("f16", 0), ("f16", 3), ("f32", 1), ("bf16", 0)])
def test_softmax_of_three_vectors_a_lane(dtype, ragged, vectors, lanes, causal):
    n = vectors * (4 if dtype == "f32" else 8) - ragged
    rows = 2048 * (64 // lanes if lanes else 1)
    if causal and ragged == 3:
        rows += 64  # (no whole number of workgroups)
    _, info, _ = _softmax(dtype, rows, n, causal, f"softmax of {rows} rows of {n} {dtype}")
    if lanes:
        assert info.vectors_per_lane == 3


@pytest.mark.parametrize("n", [129, 200, 253, 256])
def test_two_steps_of_rows_side_by_side(n):
    _softmax("f16", 16384, n, False, f"softmax of 16384 rows of {n}")
    _softmax("f16", 16448, n, True, f"causal softmax of 16448 rows of {n}")


@pytest.mark.parametrize("norm", ["layernorm", "rmsnorm"])
@pytest.mark.parametrize("dtype,n,vectors", [("f16", 1025, 3), ("f16", 1535, 3), ("f32", 640, 3), ("f16", 2049, 5), ("f16", 2639, 6), ("f32", 1024 + 4, 5), ("f32", 1791, 7),
                                             ("f16", 4095, 8), ("f32", 2048, 8)])
def test_normalisations_of_a_wave_to_a_row(dtype, n, vectors, norm):
    rows = 2050
    s = wl.ChainSpec(inputs=[(dtype, (rows, n)), (dtype, (rows, n)), (dtype, (n,)), (dtype, (n,)), (dtype, (n,))])
    v = s.op("add", s.op("add", 0, 1), 2)
    s.out(s.op("layernorm", v, 3, 4, f=[1e-5]) if norm == "layernorm" else s.op("rmsnorm", s.op("add", v, 4), 3, f=[1e-6]), dtype)
    ins = [wl.random_tensor((rows, n), dtype, 7600, scale=0.5), wl.random_tensor((rows, n), dtype, 7601, scale=0.5), wl.random_tensor((n,), dtype, 7602, scale=0.5),
           wl.random_tensor((n,), dtype, 7603, dist="positive"), wl.random_tensor((n,), dtype, 7604, scale=0.3)]
    _, info, _ = check_chain(s, ins, what=f"x + y + bias, {norm} over {n} {dtype}")
    assert info.vectors_per_lane == vectors
