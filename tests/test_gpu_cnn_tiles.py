"""The network's convolution kernels at the edges of their tiles: image sides
below a lane's eight pixels (1, 2, 3, 6), rows that end inside a step, pixel
counts that are no multiple of a step, one image and several, the narrowest
and the widest channel counts.  The comparison and its tolerances are those
of test_gpu_cnn_ops (floating-point sums against the magnitudes of their
terms)."""

import numpy as np
import pytest

import test_gpu_cnn_ops as ops
from oracle import cnn_oracle as co

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (layer index, c0, n, batch); side of the layer's output grid at its left
CASES = [
    (9, 8, 27, 1),    # 1
    (8, 8, 27, 5),    # 1, down
    (11, 8, 27, 3),   # 3, up
    (10, 8, 54, 3),   # 2
    (6, 16, 54, 1),   # 6
    (11, 16, 54, 2),  # 6, up
    (10, 8, 81, 4),   # 3
    (5, 24, 108, 1),  # 12, down
    (14, 8, 108, 1),  # 36, up
    (1, 8, 27, 1),    # 27
    (20, 32, 27, 3),  # 27, head
    (0, 32, 54, 1),   # 54, input layer
    (18, 32, 54, 1),  # 54, two 32-channel halves in
    (10, 64, 27, 2),  # 1, 512 channels
    (4, 40, 81, 1),   # 27, 80 channels
]


@pytest.mark.parametrize("op", ["forward", "dgrad", "wgrad"])
@pytest.mark.parametrize("case", CASES, ids=ops._case_id)
def test_layer_edges(case, op):
    {"forward": ops.test_layer_forward, "dgrad": ops.test_layer_dgrad, "wgrad": ops.test_layer_wgrad}[op](case)


@pytest.mark.parametrize("c0", [8, 24, 32])
def test_parameters_round_trip_and_reach_the_layers(c0):
    """set_params / get_params keep every value; the forward and the
    input-gradient copies of the weights (one launch for all layers) are those
    of the layer that owns them: a layer whose weights are zero but for one
    yields that one weight."""
    from paper_1004_1122_amd import cnn
    net = cnn.WarmStartNet(c0, seed=3)
    rng = np.random.default_rng(c0)
    vec = rng.standard_normal(net.n_params).astype(np.float32)
    net.set_params(vec)
    np.testing.assert_array_equal(net.get_params(), vec)
    n = 27
    for index, (name, kind, _, _) in enumerate(co.layer_specs(c0)):
        if kind != "conv3" or name.startswith("up") or index == 0:
            continue
        _, hi, ho, cin, cout = cnn.layer_geometry(index, n, c0)
        params = {k: [np.zeros_like(w), np.zeros_like(b)] for k, (w, b) in cnn.unpack(vec, c0).items()}
        ci, o = cin - 3, cout - 2
        params[name][0][1, 1, ci, o] = 1.5
        net.set_params(cnn.pack(params, c0))
        x = torch.zeros((1, hi, hi, cin), dtype=torch.bfloat16)
        x[0, 0, 0, ci] = 2.0
        _, yf = net.layer_forward(index, x, n)
        want = np.zeros((1, ho, ho, cout), np.float32)
        want[0, 0, 0, o] = 3.0
        np.testing.assert_array_equal(yf.cpu().numpy(), want)
        gy = torch.zeros((1, ho, ho, cout), dtype=torch.bfloat16)
        gy[0, 0, 0, o] = 2.0
        gx = net.layer_dgrad(index, gy, n).cpu().numpy()
        want = np.zeros((1, hi, hi, cin), np.float32)
        want[0, 0, 0, ci] = 3.0
        np.testing.assert_array_equal(gx, want)
