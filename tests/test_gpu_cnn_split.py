"""The fused convolution kernel multiplies on the bf16 matrix cores, each float
split in three, several pixels of a row to a column of the product: its shapes
(pixels a group, channel groups, windows that end inside a 16-byte chunk, odd
K-steps, images smaller than a tile) against 64 bits, and pixels whose value
has no split."""
import numpy as np
import pytest

import oracle
from paper_2407_18352_amd import workloads as wl
from gpu_util import parity_stats, require_gpu
from test_gpu_cnn import _run

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _workload(cin, layers, mode, S, H, W, seed=0, acts=None):
    g = np.random.default_rng(seed + 17 * cin + H * W)
    ls, c = [], cin
    for i, (cout, kh, kw) in enumerate(layers):
        m = mode[i] if isinstance(mode, list) else mode
        act = acts[i] if acts else (wl.RELU if i + 1 < len(layers) else wl.IDENTITY)
        ls.append(wl.conv_layer(900 + seed, 3 * i, c, cout, (kh, kw), mode=m, act=act))
        c = cout
    spec = {"rank": 3, "slices": [((0, 0, 0), (1, 1, 1))], "sweep": ((0, 0, 0), (S, H, W), (1, 1, 1)), "bnd": [0, 0, 0]}
    model = {"kind": "cnn", "in_channels": cin, "image": (H, W), "layers": ls}
    return wl.Workload("split", 0, "f32", [cin, c], spec, spec,
                       [g.standard_normal((S, H, W)).astype(np.float32) for _ in range(cin)],
                       [wl.sentinel_like((S, H, W)) for _ in range(c)], model)


def _both(w, path="cnn_fused_f32"):
    got, var = _run(w)
    assert var == path, var
    exp = [a.copy() for a in w.outputs]
    oracle.infer(w.in_spec, w.inputs, w.out_spec, exp, w.model)
    return np.stack([a.reshape(-1) for a in got], 1), np.stack([a.reshape(-1) for a in exp], 1)


@pytest.mark.parametrize("cin, layers, mode", [
    (4, [(8, 5, 5), (4, 3, 3)], "circular"),               # four pixels a group in both forms
    (1, [(4, 2, 2)], "zeros"),                             # one layer, 16 rows, one channel
    (3, [(12, 3, 4), (16, 2, 3), (9, 1, 5)], "replicate"), # two pixels a group; 12 and 16 channels, two groups of 4 unused
    (5, [(6, 4, 2), (13, 3, 3), (7, 2, 2), (2, 3, 1)], "zeros"),
    (8, [(8, 3, 3)], "replicate"),                         # inputs not requested ahead
    (4, [(5, 8, 8), (4, 2, 6)], "circular"),
    (4, [(4, 1, 1), (4, 7, 3), (4, 1, 2)], ["zeros", "replicate", "zeros"]),
])
@pytest.mark.parametrize("S, H, W", [(1, 37, 150), (2, 3, 5), (3, 19, 64), (1, 1, 200)])
def test_shapes_against_64_bits(cin, layers, mode, S, H, W):
    w = _workload(cin, layers, mode, S, H, W)
    got, want = _both(w)
    worst, norm, nan = parity_stats(got, want)
    # a rounding of one part in 2^24 per 8 values of K and 6 more a layer, independent; four times that for the worst
    bound = 2.0 ** -24 * np.sqrt(sum(kh * kw * c / 8 + 6 for (_, kh, kw), c in zip(layers, [cin] + [l[0] for l in layers])))
    assert nan == 0 and worst <= 16 * bound, (worst, bound)
    if H * W > 1000:
        assert norm <= bound, (norm, bound)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38])
@pytest.mark.parametrize("acts", [[1, 0], [0, 0]])
def test_values_without_a_split(value, acts):
    """One such pixel: the same classes of results as 64-bit arithmetic gives,
    everywhere else the usual accuracy (a matrix column holds neighbouring
    pixels, whose windows do not reach it)."""
    w = _workload(4, [(8, 5, 5), (4, 3, 3)], "zeros", 1, 50, 140, acts=acts)
    w.inputs[2][0, 21, 67] = value
    if value == 3e38:   # finite sums in 64 bits and in 32: weights that bring it back
        w.model["layers"][0]["W"][:, 2] *= np.float32(2.0 ** -127)
    got, want = _both(w)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fine = np.isfinite(want).all(1)
    far = np.ones((50, 140), bool)
    far[18:25, 64:71] = False                      # beyond both windows' reach of the pixel
    assert fine[far.reshape(-1)].all()
    assert parity_stats(got[fine], want[fine])[0] <= 1e-5


@pytest.mark.parametrize("exponent", [-90, -101, -120])
def test_tiny_images(exponent):
    w = _workload(4, [(8, 3, 3), (4, 3, 3)], "circular", 1, 40, 70, seed=2)
    for a in w.inputs:
        a[:] = (np.abs(a) + 0.5).astype(np.float32) * np.float32(2.0 ** exponent)
    for ly in w.model["layers"]:
        ly["b"][:] = 0
    w.model["layers"][1]["W"] *= np.float32(2.0 ** -exponent)
    got, want = _both(w)
    worst, _, nan = parity_stats(got, want)
    assert nan == 0 and worst <= 1e-5, worst


@pytest.mark.parametrize("layers, mode", [
    ([(8, 3, 3), (4, 3, 3)], "circular"), ([(8, 3, 3), (4, 3, 3)], "zeros"), ([(8, 3, 3), (4, 3, 3)], "replicate"),
    ([(6, 4, 2), (13, 3, 3), (7, 2, 2), (2, 3, 1)], "zeros"), ([(9, 2, 3), (4, 1, 5), (3, 3, 3)], ["zeros", "replicate", "zeros"])])
def test_weight_without_a_split(layers, mode):
    """The vector ALU form."""
    w = _workload(4, layers, mode, 2, 40, 70, seed=3)
    w.model["layers"][0]["W"][3, 1, 0, 1] = 2.0 ** 127
    w.inputs[1] *= np.float32(2.0 ** -126)
    got, want = _both(w, "cnn_fused_valu_f32")
    assert parity_stats(got, want)[0] <= 1e-5


@pytest.mark.parametrize("layers, H, W, path", [
    ([(4, 3, 3), (4, 2, 2)], 1536, 2048, "cnn_fused_valu_f32"), ([(4, 3, 3), (4, 2, 2)], 1535, 2048, "cnn_fused_f32"),
    ([(4, 3, 3), (4, 2, 2), (4, 1, 1)], 1536, 2048, "cnn_fused_f32")])
def test_large_images_with_few_multiplications(layers, H, W, path):
    """The vector ALU serves from 3 x 2^20 pixels on and up to 208 multiplications a
    pixel (13 x 16): both sides of the line."""
    w = _workload(4, layers, "circular", 1, H, W, seed=4)
    got, want = _both(w, path)
    assert parity_stats(got, want)[0] <= 1e-5


@pytest.mark.parametrize("layers", [[(8, 3, 3), (4, 3, 3)], [(8, 3, 3)], [(4, 3, 3)], [(4, 1, 1), (8, 3, 3), (3, 2, 2)]])
@pytest.mark.parametrize("factor, value", [(1.0e20, 1.1e25), (7.77e20, 9.3e25), (3.3e19, 5.9e24), (2.0e21, 6.1e20)])
def test_overflow_inside_a_layer(layers, factor, value):
    """One weight of 1e20 meets one pixel of 1e25 (of either sign, in a ReLU
    layer): infinite, or 0, like every output that it reaches; the other pixels
    are as accurate as ever."""
    for sign in (1, -1):
        w = _workload(4, layers, "zeros", 1, 40, 140, seed=5, acts=[1] * len(layers))
        L = w.model["layers"]
        L[0]["W"][:, 1] = 0
        L[0]["W"][2, 1, 0, 0] = factor
        for ly in L[1:]:
            ly["W"][:] = np.abs(ly["W"]) + np.float32(0.01)
        w.inputs[1][:] = 0
        w.inputs[1][0, 21, 67] = sign * np.float32(value)
        got, want = _both(w)
        assert np.isinf(want).any() == (sign > 0)
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
        rows = np.isfinite(want).all(1)
        assert np.isfinite(got[rows]).all()
        assert parity_stats(got[rows], want[rows])[0] <= 1e-5


def _fp32_error(w, got, want):
    """The worst error, in parts of the same sums without signs, over what the
    vector ALU's sums give: a rounding of one part in 2^24 per product,
    independent of each other."""
    layers = [dict(ly, W=np.abs(ly["W"]), b=np.abs(ly["b"])) for ly in w.model["layers"]]
    size = [np.zeros_like(a) for a in w.outputs]
    oracle.infer(w.in_spec, [np.abs(a) for a in w.inputs], w.out_spec, size, dict(w.model, layers=layers))
    size = np.stack([a.reshape(-1) for a in size], 1).astype(np.float64)
    terms = sum(ly["W"][0].size for ly in layers)
    return np.max(np.abs(got.astype(np.float64) - want) / size) / (2.0 ** -24 * np.sqrt(terms))


@pytest.mark.parametrize("exponent", [-112, -118, -124])
def test_tiny_hidden_values(exponent):
    """Inputs and first-layer weights of half the exponent each, the second
    layer's weights bring the sums back."""
    layers = [(8, 3, 3), (4, 3, 3)]
    w = _workload(4, layers, "circular", 1, 40, 70, seed=6)
    half = exponent // 2
    for a in w.inputs:
        a[:] = (np.abs(a) + 0.5).astype(np.float32) * np.float32(2.0 ** half)
    for ly in w.model["layers"]:
        ly["b"][:] = 0
    w.model["layers"][0]["W"] *= np.float32(2.0 ** (exponent - half))
    w.model["layers"][1]["W"] *= np.float32(2.0 ** -exponent)
    got, want = _both(w)
    assert _fp32_error(w, got, want) <= 4


@pytest.mark.parametrize("tiny", ["input", "weight", "most pixels"])
def test_tiny_factors_beside_normal_ones(tiny):
    """A channel of 2^-122 with weights that make it count, the other way round,
    and an image of 2^-122 but for one pixel."""
    layers = [(8, 3, 3), (4, 3, 3)]
    w = _workload(4, layers, "circular", 1, 40, 70, seed=7)
    L = w.model["layers"]
    if tiny == "most pixels":
        for ly in L:
            ly["b"][:] = 0
        L[1]["W"] *= np.float32(2.0 ** 122)
        for a in w.inputs:
            a[:] = (np.abs(a) + 0.5).astype(np.float32) * np.float32(2.0 ** -122)
        w.inputs[0][0, 20, 30] = 1.0
    else:
        by = np.float32(2.0 ** (-122 if tiny == "input" else 122))
        w.inputs[2] *= by
        L[0]["W"][:, 2] /= by
    got, want = _both(w)
    assert _fp32_error(w, got, want) <= 4


@pytest.mark.parametrize("cin, layers, acts", [
    (4, [(8, 5, 5), (4, 3, 3)], None), (4, [(8, 5, 5), (4, 3, 3)], [0, 0]), (3, [(4, 3, 2)], [0]), (4, [(4, 8, 8)], [1]),
    (4, [(12, 2, 7)], [0]), (8, [(8, 3, 3), (6, 2, 2), (16, 1, 1)], None), (4, [(4, 1, 1), (4, 3, 3)], [1, 1])])
@pytest.mark.parametrize("mode", ["circular", "zeros", "replicate"])
@pytest.mark.parametrize("S, H, W", [(1, 50, 140), (2, 5, 9)])
@pytest.mark.parametrize("where", ["points", "land", "with infinities"])
def test_nan_pixels(cin, layers, acts, mode, S, H, W, where):
    """NaN in single pixels, corners among them, in a third of the image, and
    beside infinities: NaN, or 0 after a ReLU, wherever a window reaches one, and
    everywhere else the usual accuracy."""
    w = _workload(cin, layers, mode, S, H, W, seed=9, acts=acts)
    if where == "land":
        w.inputs[1 % cin][:, : H // 3 + 1, : W - 3] = np.nan
    else:
        for s, y, x in ((0, 0, 0), (0, H - 1, W - 1), (0, H // 2, W // 2), (S - 1, 1, W - 2)):
            w.inputs[(y + x) % cin][s, y, x] = np.nan
    if where == "with infinities":
        w.inputs[0][S - 1, H // 2, 2] = np.inf
    got, want = _both(w)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    got, want = np.where(np.isfinite(want), got, 0), np.where(np.isfinite(want), want, 0)
    assert parity_stats(got, want)[0] <= 1e-5
