"""The network's convolution kernels at the edges of their tiles: image sides
below a lane's eight pixels (1, 2, 3, 6), rows that end inside a step, pixel
counts that are no multiple of a step, one image and several, the narrowest
and the widest channel counts.  The comparison and its tolerances are those
of test_gpu_cnn_ops (floating-point sums against the magnitudes of their
terms)."""

import pytest

import test_gpu_cnn_ops as ops

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
