"""The TV prox and the forward-backward update at the sizes and step counts where their launches
change, against the FP64 oracle: one region (64^2, 16^3) or several, the steps in one launch or
more, a launch that holds only the final primal step."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import inverse as oinv

from .helpers import gpu_context, medium, rel

pytestmark = pytest.mark.gpu

CASES = [  # dim, n, steps
    (2, 64, 63), (2, 64, 64), (2, 64, 130),           # one region: launches of 64 steps
    (2, 65, 7), (2, 65, 8), (2, 65, 9),               # several: 7 + primal in one launch, 8 | primal, 8 | 1
    (2, 97, 33),                                      # a last region of one point per axis
    (3, 16, 65), (3, 17, 3), (3, 17, 4), (3, 25, 11), (3, 49, 9), (3, 73, 4),
]


@pytest.mark.parametrize("dim, n, steps", CASES)
def test_prox_and_update_match_oracle(dim, n, steps):
    rng = np.random.default_rng(n + steps)
    draw = lambda s: (s * rng.standard_normal((n,) * dim)).astype(np.float32)  # noqa: E731
    f = np.abs(draw(1.0))
    fbar, grad = f + draw(0.1), draw(1.0)
    dev = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    f64 = lambda a: np.asarray(a, dtype=np.float64)  # noqa: E731
    with gpu_context(medium(n, d=dim), w=4, levels=5 if dim == 3 and n > 40 else 3, max_batch=1, restart=1) as ctx:
        w = ctx.tv_prox(dev(fbar), 0.3, lo=0.05, iters=steps).cpu().numpy()
        f_d, fbar_d = dev(f), dev(fbar)
        ctx.fbs_step(f_d, fbar_d, dev(grad), 0.2, 1.5, 1.7, lo=0.0, prox_iters=steps)
    # the bound of the other prox tests (single precision, errors not amplified by the projections)
    assert rel(w, oinv.tv_prox(f64(fbar), 0.3, lo=0.05, iters=steps)) < 2e-5
    f_ref, fbar_ref, _ = oinv.fbs_update(f64(f), f64(fbar), f64(grad), 0.2, 1.5, 1.7, prox_iters=steps)
    assert rel(f_d.cpu().numpy(), f_ref) < 2e-5
    assert rel(fbar_d.cpu().numpy(), fbar_ref) < 2e-5
