"""Every kernel that the network's launchers choose between, at a layer shape
that reaches it (tests/test_cnn_variants.py checks the choice on the host),
against the oracle with the tolerances of test_gpu_cnn_ops: element by element
against the sum of the magnitudes of the terms.  Batches large enough to fill
the chip hold three images in turn: the first three outputs are compared with
the oracle, the others must repeat them bit for bit, and a weight gradient is
the sum over the repeats.  Then training steps of wide networks."""

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


# (operation, layer index, c0, n, batch): kernel.  Kernels: ("patch", rows,
# channel halves), ("wave", 16-pixel tiles, 32-channel tiles), ("wgrad", columns,
# rows shorter than a step)
CASES = [
    (("forward", 1, 32, 27, 2), ("patch", 8, 1)),
    (("forward", 18, 24, 54, 1), ("patch", 8, 1)),     # 48 channels: a step spans taps
    (("forward", 4, 32, 81, 2), ("patch", 8, 2)),
    (("dgrad", 18, 40, 27, 2), ("patch", 8, 2)),       # 40 -> 80
    (("forward", 15, 32, 81, 2), ("patch", 4, 2)),     # 128 -> 64
    (("forward", 14, 32, 81, 1), ("patch", 4, 2)),     # 128 -> 64 on the upsampled grid
    (("forward", 3, 64, 81, 1), ("patch", 4, 2)),      # 128 -> 128
    (("dgrad", 3, 64, 81, 1), ("patch", 4, 2)),
    (("forward", 18, 56, 27, 2), ("patch", 4, 2)),     # 112 channels: a step spans taps
    (("dgrad", 3, 56, 81, 1), ("patch", 4, 2)),
    (("forward", 15, 56, 108, 1), ("patch", 4, 2)),    # 224 channels, side 36
    (("forward", 12, 64, 243, 1), ("wave", 1, 1)),     # 512 channels: no patch
    (("forward", 12, 40, 243, 1), ("wave", 1, 1)),     # 320 channels
    (("dgrad", 20, 64, 81, 15), ("wave", 4, 2)),       # head: one tap, 8 channels
    (("dgrad", 20, 64, 81, 9), ("wave", 2, 2)),
    (("dgrad", 20, 64, 81, 6), ("wave", 2, 1)),
    (("dgrad", 20, 64, 81, 1), ("wave", 1, 1)),
    (("forward", 20, 32, 81, 15), ("wave", 4, 1)),     # head: one tap, 32 channels
    (("forward", 20, 8, 81, 15), ("wave", 4, 1)),
    (("forward", 20, 32, 81, 9), ("wave", 2, 1)),
    (("forward", 20, 24, 81, 9), ("wave", 2, 1)),
    (("dgrad", 5, 32, 243, 15), ("wave", 4, 2)),       # transposed stride 3, 128 -> 64
    (("dgrad", 5, 32, 243, 9), ("wave", 2, 2)),
    (("dgrad", 5, 32, 243, 6), ("wave", 2, 1)),
    (("dgrad", 2, 8, 81, 15), ("wave", 4, 1)),         # transposed stride 3, 16 -> 8
    (("dgrad", 2, 24, 81, 9), ("wave", 2, 1)),
    (("forward", 2, 32, 243, 15), ("wave", 4, 2)),     # stride 3, 32 -> 64
    (("forward", 2, 40, 243, 9), ("wave", 4, 2)),      # 40 -> 80: a step spans taps
    (("forward", 2, 32, 243, 9), ("wave", 2, 2)),
    (("forward", 2, 24, 243, 9), ("wave", 2, 2)),
    (("forward", 2, 24, 243, 6), ("wave", 2, 1)),
    (("forward", 2, 32, 243, 6), ("wave", 2, 1)),
    (("forward", 2, 16, 243, 15), ("wave", 4, 1)),
    (("forward", 3, 16, 27, 1215), ("wave", 4, 1)),    # 3x3 on 9^2 images, 32 -> 32
    (("forward", 3, 16, 27, 612), ("wave", 2, 1)),
    (("forward", 3, 32, 27, 612), ("wave", 2, 2)),
    (("wgrad", 12, 64, 81, 3), ("wgrad", 64, 0)),      # 512 -> 256 on 9^2
    (("wgrad", 11, 64, 81, 3), ("wgrad", 64, 0)),      # on the upsampled grid
    (("wgrad", 8, 64, 243, 1), ("wgrad", 64, 0)),      # stride 3, 256 -> 512
    (("wgrad", 12, 40, 81, 102), ("wgrad", 64, 0)),    # two pixel splits
    (("wgrad", 9, 64, 81, 3), ("wgrad", 64, 1)),       # 3^2
    (("wgrad", 11, 64, 27, 3), ("wgrad", 64, 1)),
    (("wgrad", 8, 64, 81, 3), ("wgrad", 64, 1)),
    (("wgrad", 3, 32, 81, 18), ("wgrad", 32, 0)),      # two pixel splits
    (("wgrad", 14, 16, 81, 3), ("wgrad", 32, 0)),
    (("wgrad", 2, 24, 81, 3), ("wgrad", 32, 0)),
    (("wgrad", 20, 40, 81, 3), ("wgrad", 32, 0)),
    (("wgrad", 9, 24, 54, 6), ("wgrad", 32, 1)),
    (("wgrad", 8, 16, 81, 6), ("wgrad", 32, 1)),
    (("wgrad", 11, 16, 54, 6), ("wgrad", 32, 1)),
]


def case_id(c):
    op, index, c0, n, B = c[0]
    return f"{op}-{ops._case_id((index, c0, n, B))}"


@pytest.mark.parametrize("case", CASES, ids=case_id)
def test_kernel(case):
    from paper_1004_1122_amd import cnn
    op, index, c0, n, B = case[0]
    net, used = ops._net(c0)
    distinct = min(B, 3)
    assert B % distinct == 0
    name, x, gy, cout = ops._operands(index, c0, n, distinct, seed=300 + index)
    print("case", op, name, c0, n, B, flush=True)
    w, b = used[name]
    kind = ops._kind(name, c0)
    up = name.startswith("up")
    xin = co.up3(x) if up else x
    g = gy[..., :cout]
    xt = ops._bf16_tensor(x).repeat(B // distinct, 1, 1, 1)
    gt = ops._bf16_tensor(gy).repeat(B // distinct, 1, 1, 1)

    def repeats(t):
        for k in range(distinct, B, distinct):
            assert torch.equal(t[k:k + distinct], t[:distinct]), k
        return ops._np(t[:distinct])

    if op == "forward":
        y, yf = net.layer_forward(index, xt, n)
        ref, mag = ops._op(kind)(xin, w, b), ops._op(kind)(np.abs(xin), np.abs(w), np.abs(b))
        if kind != "conv1":
            ref = co.relu(ref)
        got = repeats(yf)
        ops._check_scaled(got, ref, mag, ops.FWD_TOL, f"{name} forward")
        np.testing.assert_array_equal(repeats(y), co.bf16(got))
    elif op == "dgrad":
        got = repeats(net.layer_dgrad(index, gt, n))
        ref = ops._op_backward(kind)(xin, w, g)[0]
        mag = ops._op_backward(kind)(np.abs(xin), np.abs(w), np.abs(g))[0]
        if up:
            ref, mag = co.up3_backward(ref), co.up3_backward(mag)
        ops._check_scaled(got, ref, mag, ops.DGRAD_TOL, f"{name} dgrad")
    else:
        grads = cnn.unpack(net.layer_wgrad(index, xt, gt, n), c0)
        _, gw, gb = ops._op_backward(kind)(xin, w, g)
        _, mw, mb = ops._op_backward(kind)(np.abs(xin), np.abs(w), np.abs(g))
        times = B // distinct
        ops._check_scaled(grads[name][0], times * gw, times * mw, ops.WGRAD_TOL, f"{name} wgrad (weights)")
        ops._check_scaled(grads[name][1], times * gb, times * mb, ops.WGRAD_TOL, f"{name} wgrad (bias)")
    net.drop_workspaces()


@pytest.mark.parametrize("c0,n", [(32, 81), (24, 27)])
def test_training_step_of_wide_networks(c0, n):
    """Gradients and loss of one step, whose input gradients pass through the
    masked store, the added skip gradient and the FP32 skip split.  Each output
    channel takes one input channel at one tap with weight 1 (the FP32 head takes
    all), and biases and inputs are multiples of 1/4, so every activation is exact
    in bfloat16 and the ReLU masks are the oracle's (with dense weights a few activations round
    to the other side and move the gradients of such a network by percents).
    The gradients are then held to the layers' bar: 1e-4 of the sum of the
    magnitudes of their terms."""
    from paper_1004_1122_amd import cnn
    B = 2
    rng = np.random.default_rng(c0)
    params = {}
    for name, kind, cin, cout in co.layer_specs(c0):
        w = np.ones((cin, cout)) if kind == "conv1" else np.zeros((3, 3, cin, cout))
        if kind != "conv1":
            for out, c in enumerate(rng.permutation(np.resize(rng.permutation(cin), cout))):
                w[(*rng.integers(0, 3, size=2), c, out)] = 1.0
        params[name] = [w, rng.integers(-1, 2, size=cout) * 0.25]
    net = cnn.WarmStartNet(c0, params=cnn.pack(params, c0))
    phase = (rng.random((B, n, n)) < 0.5).astype(np.uint8)
    x = np.stack([phase.astype(np.float64), np.ones(phase.shape)], axis=-1)
    tgt = rng.standard_normal((B, 2, n, n)) * 0.3
    loss = net.train_step(phase, np.full(B, 4.0, np.float32), torch.from_numpy(tgt), update=False)
    got = cnn.unpack(net.get_grads(), c0)
    y, acts = co.forward(params, x, c0)
    assert all(np.array_equal(a, co.bf16(a)) for k, a in acts.items() if k != "head")
    ref_loss, gy = co.rel_mse(y, np.moveaxis(tgt - np.array([1.0, 0.0])[None, :, None, None], 1, -1))
    assert loss == pytest.approx(ref_loss, rel=1e-6)
    ref = co.backward(params, acts, gy, c0, round_grad=co.bf16)
    mag = co.backward(params, acts, np.abs(gy), c0, round_grad=co.bf16)
    for name in params:
        assert np.any(ref[name][0]), name
        for k in (0, 1):
            ops._check_scaled(got[name][k], ref[name][k], mag[name][k], ops.WGRAD_TOL, f"{name}[{k}]")
