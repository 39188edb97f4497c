"""NaN and infinities: they stay with their right-hand side, and the TV prox treats them as the
formula with fmax does (a NaN primal value becomes the bound)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth

from .helpers import gpu_context, medium, rel, to_dev

pytestmark = pytest.mark.gpu

BAD = {1: complex(np.nan, 0.0), 4: complex(np.inf, -np.inf)}  # right-hand side: value at one point


def poisoned(r):
    out = r.clone()
    for b, v in BAD.items():
        out[b].view(-1)[out[b].numel() // 2 + b // 2] = v  # inside the interior
    return out


def check(clean, bad):
    for b in range(clean.shape[0]):
        if b in BAD:
            assert not bool(torch.isfinite(torch.view_as_real(bad[b])).all()), b
        else:
            assert bool((bad[b] == clean[b]).all()), b


# the coarse levels in one launch (11^2 below), in two (12^2, 8^3), the coarsest grid alone (25^2, 9^3)
@pytest.mark.parametrize("n, levels, d", [(25, 3, 2), (29, 3, 2), (33, 2, 2), (13, 3, 3), (17, 3, 3)])
def test_cycle_keeps_right_hand_sides_apart(n, levels, d):
    with gpu_context(medium(n, seed=5, d=d), levels=levels, max_batch=6, restart=1, cycle=3) as ctx:
        r = to_dev(synth.complex_field((6, *ctx.grid_shape()), 40))
        check(ctx.precondition(r), ctx.precondition(poisoned(r)))
        c = to_dev(synth.complex_field((6, *(ctx.info.coarsest_n,) * d), 41))
        check(ctx.coarse_solve(c), ctx.coarse_solve(poisoned(c)))


@pytest.mark.parametrize("n, d", [(11, 2), (5, 3)])
def test_sensor_products_keep_right_hand_sides_apart(n, d):
    sens = np.random.default_rng(1).choice([-1.0, 1.0], (19, d)) * (n + np.arange(19)[:, None])
    with gpu_context(medium(n, seed=5, d=d), w=4, levels=2, max_batch=6, restart=1) as ctx:
        ctx.farfield_set(sens)
        u = to_dev(synth.complex_field((6, *ctx.grid_shape()), 42))
        check(ctx.farfield(u), ctx.farfield(poisoned(u)))
        r = to_dev(synth.complex_field((6, 19), 43))
        for clean, bad in zip(ctx.farfield_adjoint(r), ctx.farfield_adjoint(poisoned(r))):
            check(clean, bad)


def prox_reference(v, lam, lo, iters):
    """FGP in FP64 with the non-finite rules of fmax: a NaN loses against the bound and against 1."""
    dim = v.ndim
    p = np.zeros((dim, *v.shape))
    r = np.zeros_like(p)
    t = 1.0

    def primal(q):
        dt = np.zeros_like(v)
        for a in range(dim):
            low = [slice(None)] * dim
            high = [slice(None)] * dim
            low[a], high[a] = slice(0, -1), slice(1, None)
            dt[tuple(high)] += q[a][tuple(low)]
            dt[tuple(low)] -= q[a][tuple(low)]
        return np.fmax(v - lam * dt, lo)

    for _ in range(iters):
        w = primal(r)
        g = np.zeros_like(p)
        for a in range(dim):
            low = [slice(None)] * dim
            low[a] = slice(0, -1)
            g[a][tuple(low)] = np.diff(w, axis=a)
        q = r + g / (4 * dim * lam)
        q = q * (1.0 / np.fmax(1.0, np.sqrt((q ** 2).sum(axis=0))))
        tn = 0.5 * (1 + np.sqrt(1 + 4 * t * t))
        r = q + (t - 1) / tn * (q - p)
        p, t = q, tn
    return primal(p)


# one region; several, with the values on their borders and in their halos
@pytest.mark.parametrize("shape, steps", [((40, 40), 20), ((120, 120), 20), ((12,) * 3, 9), ((29,) * 3, 9)])
def test_prox(shape, steps):
    v = np.random.default_rng(len(shape)).standard_normal(shape).astype(np.float32)
    n = shape[0]
    flat = v.reshape(-1)
    spots = np.random.default_rng(2).choice(flat.size, 12, replace=False)
    spots[:2] = 0, flat.size - 1  # corners of the grid
    flat[spots[0::3]] = np.nan
    flat[spots[1::3]] = np.inf
    flat[spots[2::3]] = -np.inf
    v[(min(47, n - 1),) * v.ndim] = np.nan  # the last point of the first region (2D)
    with gpu_context(medium(n, d=v.ndim), w=4, levels=3, max_batch=1, restart=1) as ctx:
        w = ctx.tv_prox(torch.tensor(v, device="cuda"), 0.3, lo=0.05, iters=steps).cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = prox_reference(v.astype(np.float64), 0.3, np.float32(0.05).astype(np.float64), steps)
    assert not np.isnan(ref).any() and np.array_equal(np.isinf(w), np.isinf(ref)) and not np.isnan(w).any()
    ok = np.isfinite(ref)
    assert rel(w[ok], ref[ok]) < 2e-5  # the bound of the other prox tests
