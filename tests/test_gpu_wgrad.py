"""Weight and bias gradients of the networks at the edges of their pixel tiles (8 or 4 rows of 32)
and planes, against the FP64 reference."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import learned, learned3d

from .helpers import rel

pytestmark = pytest.mark.gpu


def bf16_round(a):
    return torch.tensor(a, dtype=torch.float32).to(torch.bfloat16).to(torch.float64).numpy()


# one tile, one pixel or row more, remainders at every level, more tiles than a block takes at once
@pytest.mark.parametrize("shape", [(1, 8, 32), (2, 9, 33), (3, 3, 31), (1, 17, 64), (40, 66, 70),
                                   (1, 1, 8, 32), (2, 3, 9, 33), (1, 5, 4, 31)])
def test_edge_gradients_match_reference(shape):
    from paper_2107_03679_amd import helm

    dim = len(shape) - 1
    ref = learned if dim == 2 else learned3d
    p = {k: bf16_round(v) if k.endswith(".w") else v for k, v in ref.init_params(3).items()}
    rng = np.random.default_rng(sum(shape))
    for k in p:
        if k.endswith(".b"):
            p[k] = 0.1 * rng.standard_normal(p[k].shape)
    x = bf16_round(rng.standard_normal((*shape, 4)))
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")  # noqa: E731
    net = helm.Net(seed=0, dim=dim)
    net.set_params(p)
    y, t = ref.forward(p, x)
    # the loss sees only the last pixel along each axis: what an edge drops is not hidden by the rest
    gy = np.zeros_like(y)
    for a in range(1, 1 + dim):
        sl = [slice(None)] * (2 + dim)
        sl[a] = -1
        gy[tuple(sl)] = 1.0
    out = net.forward(dev(x))
    net.backward(dev(x), out - dev(gy))
    grads, want = net.grads(), ref.backward(p, t, gy / shape[0])
    net.close()
    for name, g in want.items():
        # BF16 activations and gradients through up to 15 layers: the bound of the other gradient tests
        assert rel(grads[name], g) < 0.1, (name, rel(grads[name], g))


def test_batch_gradient_is_the_sum_of_its_images():
    """Images share no taps: a batch's gradient is the mean of its images' (the loss is per image)."""
    from paper_2107_03679_amd import helm

    net = helm.Net(seed=4)
    x = torch.randn((3, 19, 45, 4), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    tgt = torch.zeros((3, 19, 45, 2), device="cuda")
    net.backward(x, tgt)
    whole = net.grads()
    parts = []
    for i in range(3):
        net.backward(x[i:i + 1], tgt[i:i + 1])
        parts.append(net.grads())
    net.close()
    for name, g in whole.items():
        # each image's gradient enters the batch scaled by 1/3 before its BF16 rounding: 2^-9 of it
        assert rel(sum(q[name].astype(np.float64) for q in parts) / 3, g.astype(np.float64)) < 1e-2, name
