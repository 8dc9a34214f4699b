"""Fully connected layers on few images (32 images and 64 outputs a block, a K
range over four waves) and max-pools that share their channels between the
lanes of a window, against the oracle: edges of tiles, K not a multiple of a
step or of four floats, padded ranges, channel counts that leave lanes idle."""
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


def _both(S, H, W, layers, n_out, seed):
    g = np.random.default_rng(seed)
    spec = {"rank": 3, "slices": [((0, 0, 0), (1, 1, 1))], "sweep": ((0, 0, 0), (S, H, W), (1, 1, 1)), "bnd": [0, 0, 0]}
    w = wl.Workload("layers_split", 0, "f32", [1, n_out], spec, wl.pointwise_spec(S),
                    [g.standard_normal((S, H, W)).astype(np.float32)], [wl.sentinel_like((S,)) for _ in range(n_out)],
                    {"kind": "cnn", "in_channels": 1, "image": (H, W), "layers": layers})
    got, var = _run(w)
    assert var == "cnn_layers_f32", var
    exp = [a.copy() for a in w.outputs]
    oracle.infer(w.in_spec, w.inputs, w.out_spec, exp, w.model)
    return np.stack([a.reshape(-1) for a in got], 1), np.stack([a.reshape(-1) for a in exp], 1)


@pytest.mark.parametrize("S, H, W, out", [
    (1, 16, 16, 17), (31, 16, 16, 64), (33, 16, 17, 65), (100, 17, 19, 33), (1, 29, 40, 256), (1024, 17, 19, 33),
    (100, 29, 40, 256), (1400, 16, 31, 128), (2720, 13, 21, 64), (4096, 16, 16, 17), (4097, 16, 16, 17)])   # the last by the 128-image kernel
def test_linear(S, H, W, out):
    layers = [wl.linear_layer(61, 0, H * W, out), wl.linear_layer(62, 0, out, 3, act=0)]
    got, want = _both(S, H, W, layers, 3, seed=S + out)
    worst, norm, nan = parity_stats(got, want)
    # sums of H W + out products, each rounded to 2^-24 of a partial sum: at most a random walk of that many roundings
    bound = 2.0 ** -24 * np.sqrt(H * W + out)
    assert nan == 0 and worst <= 8 * bound and norm <= bound, (worst, norm, bound)


@pytest.mark.parametrize("pool", [(1, 1), (1, 2), (2, 2), (1, 3), (2, 3), (4, 2), (3, 3), (4, 4)])
@pytest.mark.parametrize("cout", [1, 3, 6, 8, 11, 16])
def test_pool_lanes(pool, cout):
    H, W = 25, 27
    h, w_ = (24 - pool[0]) // pool[0] + 1, (25 - pool[1]) // pool[1] + 1
    layers = [wl.conv_layer(63, 0, 1, cout, (2, 3), padding="valid", act=cout % 2), {"kind": "pool", "kernel": pool},
              wl.linear_layer(64, 0, h * w_ * cout, 2, act=0)]
    got, want = _both(5, H, W, layers, 2, seed=cout)
    worst, norm, nan = parity_stats(got, want)
    bound = 2.0 ** -24 * np.sqrt(h * w_ * cout + 6)
    assert nan == 0 and worst <= 8 * bound, (worst, bound)
