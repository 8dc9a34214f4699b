"""The fp32 fused kernels multiply on the bf16 matrix cores, each float split
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


def _run(w, path="mlp_f32_h"):
    got, var = run_infer(w)
    assert var.startswith(path), var
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


@pytest.mark.parametrize("dims", [
    [5, 129, 1], [16, 1000, 5], [48, 300, 8],                 # one hidden layer: one and three K-steps, two output groups
    [9, 200, 50, 1], [16, 257, 32, 4], [17, 160, 64, 5],      # two: one and two blocks of the second a pass
    [9, 5, 300, 2], [1, 33, 225, 1],                          # several passes, the last with an empty block
    [9, 400, 64, 1], [20, 129, 65, 3],                        # lo parts in global memory
    [9, 40, 512, 1], [14, 64, 512, 1]])                       # eight passes
@pytest.mark.parametrize("n", [1, 33, 3001, 4096, 4097, 70001])
def test_any_widths_against_64_bits(dims, n):
    g = np.random.default_rng(sum(dims) + n)
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    got, want = _run(w, "mlp_f32w")
    worst, norm, nan = parity_stats(got, want)
    assert nan == 0 and worst <= 4 * 4 * _bound(dims), (dims, worst, _bound(dims))
    if n > 1000:
        assert norm <= _bound(dims), (dims, norm, _bound(dims))


@pytest.mark.parametrize("acts", [[0, 0, 0], [0, 1, 1], [1, 0, 0]])
def test_any_widths_activations_and_window(acts):
    """Identity hidden layers, a ReLU output layer, a clamped 3 x 3 window on a
    grid narrower than a tile, outputs shifted along a periodic dimension."""
    g = np.random.default_rng(5)
    ny, nx = 37, 19
    fields = [g.standard_normal((ny, nx)).astype(np.float32) for _ in range(3)]
    spec = {"rank": 2, "slices": [((-1, -1), (3, 3))], "sweep": ((0, 0), (ny, nx), (1, 1)), "bnd": [wl.CLAMP, wl.PERIODIC]}
    ospec = {"rank": 2, "slices": [((0, 2), (1, 1))], "sweep": ((0, 0), (ny, nx), (1, 1)), "bnd": [wl.NONE, wl.PERIODIC]}
    w = wl.Workload("split", 0, "f32", [27, 170, 40, 2], spec, ospec, fields, [wl.sentinel_like((ny, nx)) for _ in range(2)])
    w.model = wl.make_model(91, w.dims, "f32")
    w.model["act"] = acts
    got, var = run_infer(w)
    exp = [o.copy() for o in w.outputs]
    oracle.scatter(ospec, exp, oracle.infer_rows(spec, fields, w.model))
    worst, _, nan = parity_stats(np.stack([a.reshape(-1) for a in got], 1), np.stack([a.reshape(-1) for a in exp], 1))
    assert nan == 0 and worst <= 1e-5, (var, worst)


@pytest.mark.parametrize("dims", [[5, 64, 64, 1], [9, 128, 128, 128, 1], [20, 128, 128, 5], [9, 200, 50, 1], [5, 300, 6]])
def test_infinities_and_their_neighbours(dims):
    """Infinite and NaN inputs in some points: the same classes of results as
    64-bit arithmetic gives them, and every other point (some in the same wave)
    as accurate as ever."""
    n = 201
    g = np.random.default_rng(dims[0])
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    for k, v in ((3, np.inf), (40, -np.inf), (41, np.nan), (130, np.inf), (200, -np.inf)):
        w.inputs[k % dims[0]][k] = v
    got, want = _run(w, "mlp_")
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fine = np.isfinite(want).all(1)
    assert fine.sum() >= n - 5
    assert parity_stats(got[fine], want[fine])[0] <= 1e-5


@pytest.mark.parametrize("exponent", [127, 126, -90, -99, -101, -120])
@pytest.mark.parametrize("dims", [[7, 64, 64, 2], [12, 128, 128, 1], [12, 200, 40, 1]])
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
    got, want = _run(w, "mlp_")
    assert np.isfinite(want).all()
    worst, _, nan = parity_stats(got, want)
    assert nan == 0 and worst <= 1e-5, worst


@pytest.mark.parametrize("value", [2.0 ** 127, 3e38])
@pytest.mark.parametrize("dims", [[6, 128, 128, 1], [6, 200, 70, 1]])
def test_weight_without_a_split(value, dims):
    """One first-layer weight of 2^127 and more, met by inputs of 2^-127."""
    n = 100
    g = np.random.default_rng(11)
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(6)])
    w.inputs[2] = (w.inputs[2] * np.float32(2.0 ** -120) * np.float32(2.0 ** -6)).astype(np.float32)
    w.model["W"][0][17, 2] = value
    got, want = _run(w, "mlp_")
    assert parity_stats(got, want)[0] <= 1e-5


@pytest.mark.parametrize("factor, value", [(1.0e20, 1.1e25), (7.77e20, 9.3e25), (3.3e19, 5.9e24), (2.0e21, 6.1e20)])
@pytest.mark.parametrize("dims", [[7, 64, 1], [7, 64, 64, 2], [12, 128, 128, 128, 1], [12, 40, 1], [12, 200, 40, 1], [9, 300, 3]])
def test_overflow_inside_a_layer(dims, factor, value):
    """One weight of 1e20 meets one input of 1e25 in some points, everything else
    is of order 1: the neuron is infinite (or, negative, 0 after its ReLU) and
    so is every output that it reaches; the other points are as accurate as ever."""
    n = 100
    g = np.random.default_rng(dims[0])
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    W = w.model["W"]
    W[0][:, 3] = 0
    W[0][17, 3] = factor
    for l in range(1, len(W)):
        W[l][:] = np.abs(W[l]) + np.float32(0.01)   # the infinity reaches every output, and meets no other sign
    w.inputs[3][:] = 0
    for k, sign in ((5, 1), (37, -1), (64, 1), (90, -1), (99, 1)):
        w.inputs[3][k] = sign * np.float32(value) * np.float32(1 + 0.01 * k)
    got, want = _run(w, "mlp_")
    assert np.array_equal(np.isinf(want).all(1), np.isin(np.arange(n), [5, 64, 99]))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fine = np.isfinite(want)
    assert np.isfinite(got[fine]).all()
    rows = fine.all(1)
    assert parity_stats(got[rows], want[rows])[0] <= 1e-5


def _fp32_error(w, got, want):
    """The worst error, in parts of the same sums without signs, over what the
    fp32 instruction's sums give: a rounding of one part in 2^24 per product,
    independent of each other."""
    m = dict(w.model, W=[np.abs(x) for x in w.model["W"]], b=[np.abs(x) for x in w.model["b"]])
    size = oracle.infer_rows(w.in_spec, [np.abs(x) for x in w.inputs], m).astype(np.float64)
    return np.max(np.abs(got.astype(np.float64) - want) / size) / (2.0 ** -24 * np.sqrt(sum(w.dims[:-1])))


@pytest.mark.parametrize("exponent", [-105, -112, -118, -124])
@pytest.mark.parametrize("dims", [[7, 64, 64, 2], [7, 64, 64, 64, 1], [12, 128, 128, 1], [12, 200, 40, 1]])
def test_tiny_hidden_values(dims, exponent):
    """First-layer weights and inputs of half the exponent each make hidden
    values of 2^exponent, the next layer's weights bring them back."""
    n = 300
    g = np.random.default_rng(-exponent)
    half = exponent // 2
    w = _workload(dims, n, [(g.uniform(0.5, 1, n) * 2.0 ** half).astype(np.float32) for _ in range(dims[0])])
    w.model["b"] = [np.zeros_like(b) for b in w.model["b"]]
    w.model["W"][0] = (w.model["W"][0] * np.float32(2.0 ** (exponent - half))).astype(np.float32)
    w.model["W"][1] = (w.model["W"][1] * np.float32(2.0 ** -exponent)).astype(np.float32)
    got, want = _run(w, "mlp_")
    assert _fp32_error(w, got, want) <= 4


@pytest.mark.parametrize("tiny", ["input", "weight"])
@pytest.mark.parametrize("dims", [[7, 64, 64, 2], [12, 128, 128, 1], [12, 200, 40, 1], [12, 300, 1]])
def test_one_tiny_factor_beside_normal_ones(dims, tiny):
    """A feature of 2^-122 with first-layer weights that make it count as much as
    the others, or the other way round."""
    n = 300
    g = np.random.default_rng(len(dims))
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    by = np.float32(2.0 ** (-122 if tiny == "input" else 122))
    w.inputs[2] = (w.inputs[2] * by).astype(np.float32)
    w.model["W"][0][:, 2] = (w.model["W"][0][:, 2] / by).astype(np.float32)
    got, want = _run(w, "mlp_")
    assert _fp32_error(w, got, want) <= 4


@pytest.mark.parametrize("dims", [[9, 200, 50, 1], [5, 300, 6], [9, 5, 300, 2], [20, 129, 65, 3], [5, 50, 50, 1], [9, 100, 70, 90, 3]])
def test_infinities_through_identity_layers(dims):
    """An infinite feature whose weights are all positive makes every neuron of
    an identity layer +inf or -inf: outputs infinite, and none of them NaN from
    neurons that the kernel pads its blocks with."""
    n = 201
    g = np.random.default_rng(dims[0] + 1)
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    w.model["act"] = [wl.IDENTITY] * (len(dims) - 1)
    w.model["W"] = [np.abs(x) + np.float32(1e-3) for x in w.model["W"]]
    for k, v in ((3, np.inf), (40, -np.inf), (130, np.inf), (200, -np.inf)):
        w.inputs[k % dims[0]][k] = v
    got, want = _run(w, "mlp_")
    assert np.isinf(want[[3, 40, 130, 200]]).all() and np.isfinite(want).all(1).sum() == n - 4
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fine = np.isfinite(want).all(1)
    assert parity_stats(got[fine], want[fine])[0] <= 1e-5


@pytest.mark.parametrize("form", ["split", "plain", "behind"])
@pytest.mark.parametrize("dims", [
    [9, 128, 128, 128, 1], [36, 128, 128, 4], [64, 128, 1], [17, 64, 64, 5], [36, 64, 64, 64, 64, 64, 64, 8], [5, 50, 30, 1],
    [5, 300, 6], [48, 300, 1], [9, 200, 30, 1], [17, 160, 64, 5], [9, 400, 64, 1], [20, 129, 65, 3]])
def test_fp32_path_in_each_weight_form(dims, form):
    """Every tile on the fp32 instruction: a point with an infinite input in each
    (weights put together from their parts), a weight that has no split (fp32
    weights in the image), a tiny weight that meets a large input (fp32 weights
    behind it)."""
    n = 500
    g = np.random.default_rng(sum(dims))
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    if form == "split":
        w.inputs[1][::17] = np.inf
    elif form == "plain":
        w.inputs[2][:] = (w.inputs[2] * np.float32(2.0 ** -126)).astype(np.float32)
        w.model["W"][0][11, 2] = 2.0 ** 127
    else:
        w.inputs[2][:] = (w.inputs[2] * np.float32(2.0 ** 122)).astype(np.float32)
        w.model["W"][0][:, 2] = (w.model["W"][0][:, 2] * np.float32(2.0 ** -122)).astype(np.float32)
    got, want = _run(w, "mlp_")
    rows = np.isfinite(w.inputs[1])
    w.inputs = [x[rows] for x in w.inputs]
    w.in_spec = wl.pointwise_spec(int(rows.sum()))
    assert _fp32_error(w, got[rows], want[rows]) <= 4


@pytest.mark.parametrize("dims", [[9, 300, 40, 2], [12, 160, 7], [9, 40, 512, 1]])
def test_any_widths_without_allocation(dims):
    """The same kernel, and the same bits, through hpacml_infer_noalloc; on maps
    outside the 32-bit form (one input strided) both take the other paths."""
    import torch
    from paper_2407_18352_amd import _abi, api
    n = 5000
    g = np.random.default_rng(dims[1])
    w = _workload(dims, n, [g.uniform(-1, 1, n).astype(np.float32) for _ in range(dims[0])])
    want = oracle.infer_rows(w.in_spec, w.inputs, w.model)
    m = api.Model(w.model)
    for strided in (False, True):
        ins = [torch.from_numpy(a).cuda() for a in w.inputs]
        if strided:
            ins[1] = torch.stack([ins[1], ins[1]], 1)[:, 0]
        got = []
        for noalloc in (False, True):
            outs = [torch.zeros(n, device="cuda") for _ in range(dims[-1])]
            mi, mo = api.Map(w.in_spec, ins, _abi.TO), api.Map(w.out_spec, outs, _abi.FROM)
            assert api.variant(m, mi, mo) == ("mlp_layers_f32" if strided else "mlp_f32w")
            if noalloc:
                st = torch.cuda.current_stream().cuda_stream
                assert _abi.lib().hpacml_infer_noalloc(m.handle, mi.handle, mo.handle, st) == _abi.OK
            else:
                api.infer(m, mi, mo)
            torch.cuda.synchronize()
            got.append(np.stack([o.cpu().numpy() for o in outs], 1))
            assert parity_stats(got[-1], want)[0] <= 1e-5
            mi.close(), mo.close()
        if not strided:
            assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
    m.close()
