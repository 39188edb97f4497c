"""Weight and bias gradients bit for bit: networks whose activations and gradients are all exact in
BF16 and whose sums are exact in single precision, so that the FP64 reference is the answer."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import learned, learned3d

pytestmark = pytest.mark.gpu


def _exact(a, dtype):
    return np.array_equal(torch.tensor(a).to(dtype).to(torch.float64).numpy(), a)


def problem(shape, monkeypatch):
    """Every output channel is an input channel at one tap, where two inputs are concatenated one of
    each (in 3D of either), the last layer's the sum of eight; the input is sparse in {0, 1}, and so
    is the loss gradient, in {-1, 0, 1}: pooled values are small multiples of a power of two.  Checked
    on the way through the reference."""
    dim = len(shape) - 1
    ref = learned if dim == 2 else learned3d
    back = "conv3x3_backward" if dim == 2 else "conv_backward"
    rng = np.random.default_rng(sum(shape))
    up = {"B2": ref.CH[3], "B1": ref.CH[2], "B0": ref.CH[1]}
    p = {}
    for name, cin, cout, _ in ref.LAYERS:
        w = np.zeros((3,) * dim + (cin, cout))

        def one(ci, co):
            w[tuple(rng.choice([0, 1, 1, 2], dim)) + (ci, co)] = 1.0

        if name == "O":
            for ci, co in enumerate(rng.permutation(np.repeat([0, 1], cin // 2))):
                one(ci, co)
        elif name in up:
            from_up, skip = rng.permutation(up[name]), up[name] + rng.permutation(cin - up[name])
            for co in range(cout):
                if dim == 2 or co % 2:
                    one(from_up[co % len(from_up)], co)
                if dim == 2 or not co % 2:
                    one(skip[co % len(skip)], co)
        else:
            for co, ci in enumerate(rng.permutation(np.arange(cout) % cin)):
                one(ci, co)
        p[name + ".w"], p[name + ".b"] = w, np.zeros(cout)
    x = (rng.random((*shape, 4)) < (0.5 if dim == 2 else 0.25)).astype(np.float64)
    y, t = ref.forward(p, x)
    gy = (rng.random(y.shape) < (0.01 if dim == 2 else 0.001)) * rng.choice([-1.0, 1.0], y.shape)
    for a in range(1, 1 + dim):  # and the last pixel along each axis
        sl = [slice(None)] * (2 + dim)
        sl[a] = -1
        gy[tuple(sl)] = rng.random(gy[tuple(sl)].shape) < (0.1 if dim == 2 else 0.01)
    assert shape[0] & (shape[0] - 1) == 0  # the loss is divided by the images
    orig = getattr(ref, back)

    def checked(xx, w, g):
        assert _exact(xx, torch.bfloat16) and _exact(g, torch.bfloat16)
        out = orig(xx, w, g)
        assert _exact(out[1], torch.float32) and _exact(out[2], torch.float32)
        return out

    monkeypatch.setattr(ref, back, checked)
    want = ref.backward(p, t, gy / shape[0])
    return p, x, y, gy, want


SHAPES = [(1, 8, 32), (2, 9, 33), (4, 3, 31), (1, 17, 64), (32, 66, 70), (1, 5, 9, 33), (1, 4, 9, 34),
          (1, 6, 17, 33), (2, 9, 16, 40)]


@pytest.mark.parametrize("shape", SHAPES)
def test_gradients_are_exact(shape, monkeypatch):
    from paper_2107_03679_amd import helm

    p, x, y, gy, want = problem(shape, monkeypatch)
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")  # noqa: E731
    net = helm.Net(seed=0, dim=len(shape) - 1)
    net.set_params(p)
    assert np.array_equal(net.forward(dev(x)).cpu().numpy(), y)
    net.backward(dev(x), dev(y - gy))
    grads = net.grads()
    net.close()
    for name, g in want.items():
        assert np.array_equal(grads[name], g), name
