"""The fp32 fused kernel multiplies on the bf16 matrix cores, each float split
in three: its shapes (K-steps of the first layer, layers whose smallest parts
stay in global memory, groups of four outputs), values that have no split, and
its error against 64 bits."""
import numpy as np
import pytest

import oracle
from paper_2407_18352_amd import workloads as wl
from gpu_util import parity_stats, require_gpu, run_infer

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _workload(dims, n, inputs, seed=3):
    spec = wl.pointwise_spec(n)
    w = wl.Workload("split", 0, "f32", dims, spec, spec, inputs, [wl.sentinel_like((n,)) for _ in range(dims[-1])])
    w.model = wl.make_model(70 + seed, dims, "f32")
    return w


def _run(w):
    got, var = run_infer(w)
    assert var.startswith("mlp_f32_h"), var
    return np.stack(got, 1), oracle.infer_rows(w.in_spec, w.inputs, w.model)


# sums of K products rounded to 24 bits: one part in 2^24 per rounding, K / 16 + 6
# roundings a layer, independent of each other; four times that for the worst value
def _bound(dims):
    return 2.0 ** -24 * np.sqrt(sum(d / 16 + 6 for d in dims[:-1]))


@pytest.mark.parametrize("dims", [
    [1, 64, 1], [16, 64, 64, 4], [17, 64, 64, 5], [64, 64, 64, 64, 64, 64, 64, 64, 8],   # the last: lo parts in global memory
    [16, 128, 1], [32, 128, 128, 3], [33, 128, 128, 8], [49, 128, 128, 4],
    [9, 128, 128, 128, 1], [36, 128, 128, 128, 8]])                                        # lo parts in global memory
@pytest.mark.parametrize("n", [1, 33, 3001])
def test_shapes_against_64_bits(dims, n):
    g = np.random.default_rng(sum(dims) + n)
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    got, want = _run(w)
    worst, norm, nan = parity_stats(got, want)
    assert nan == 0 and worst <= 4 * 4 * _bound(dims), (dims, worst, _bound(dims))
    if n > 1000:
        assert norm <= _bound(dims), (dims, norm, _bound(dims))


@pytest.mark.parametrize("dims", [[5, 64, 64, 1], [9, 128, 128, 128, 1], [20, 128, 128, 5]])
def test_infinities_and_their_neighbours(dims):
    """Infinite and NaN inputs in some points: the same classes of results as
    64-bit arithmetic gives them, and every other point (some in the same wave)
    as accurate as ever."""
    n = 201
    g = np.random.default_rng(dims[0])
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    for k, v in ((3, np.inf), (40, -np.inf), (41, np.nan), (130, np.inf), (200, -np.inf)):
        w.inputs[k % dims[0]][k] = v
    got, want = _run(w)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fine = np.isfinite(want).all(1)
    assert fine.sum() >= n - 5
    assert parity_stats(got[fine], want[fine])[0] <= 1e-5


@pytest.mark.parametrize("exponent", [127, 126, -90, -99, -101, -120])
@pytest.mark.parametrize("dims", [[7, 64, 64, 2], [12, 128, 128, 1]])
def test_ends_of_the_range(dims, exponent):
    """Inputs of 2^exponent with first-layer weights that bring them back, and
    no biases: the points keep 24 bits whether or not their inputs split."""
    n = 70
    g = np.random.default_rng(exponent + 200)
    scale = np.float32(2.0 ** exponent)
    w = _workload(dims, n, [(g.uniform(1, 1.99, n).astype(np.float32) * scale) for _ in range(dims[0])])
    w.model["b"] = [np.zeros_like(b) for b in w.model["b"]]
    if exponent > 0:
        w.model["W"][0] = (w.model["W"][0] * np.float32(2.0 ** -100)).astype(np.float32)
        w.model["W"][0] = (w.model["W"][0] * np.float32(2.0 ** (100 - exponent))).astype(np.float32)
    else:
        w.model["W"][-1] = (w.model["W"][-1] * np.float32(2.0 ** -exponent)).astype(np.float32)
    got, want = _run(w)
    assert np.isfinite(want).all()
    worst, _, nan = parity_stats(got, want)
    assert nan == 0 and worst <= 1e-5, worst


@pytest.mark.parametrize("value", [2.0 ** 127, 3e38])
def test_weight_without_a_split(value):
    """One first-layer weight of 2^127 and more, met by inputs of 2^-127."""
    dims, n = [6, 128, 128, 1], 100
    g = np.random.default_rng(11)
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(6)])
    w.inputs[2] = (w.inputs[2] * np.float32(2.0 ** -120) * np.float32(2.0 ** -6)).astype(np.float32)
    w.model["W"][0][17, 2] = value
    got, want = _run(w)
    assert parity_stats(got, want)[0] <= 1e-5
