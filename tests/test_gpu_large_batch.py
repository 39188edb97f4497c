"""Batches beyond 65536 right-hand sides, the end of a grid's second dimension: equal to the small
batch they repeat."""
from __future__ import annotations

import numpy as np
import pytest

import synth

from .helpers import gpu_context, medium, to_dev

pytestmark = pytest.mark.gpu

REP, B = 1025, 64  # 65600 right-hand sides


def test_sensor_adjoint():
    sens = np.array([[6.0, 0.5], [-1.0, -7.0], [0.3, 8.0]])
    r = to_dev(synth.complex_field((B, 3), 20))
    with gpu_context(medium(5, seed=2), w=1, levels=2, max_batch=B, restart=1) as ctx:
        ctx.farfield_set(sens)
        want = ctx.farfield_adjoint(r)
        got = ctx.farfield_adjoint(r.repeat(REP, 1))
        for a, b in zip(got, want):
            assert bool((a.view(REP, *b.shape) == b).all())


def test_coarse_levels_in_two_launches():
    """A 12^2 coarsest grid (144 points) below 45^2 and 23^2."""
    nmap = medium(29, seed=2)
    with gpu_context(nmap, levels=3, max_batch=B, restart=1) as ctx:
        assert ctx.info.coarsest_n == 12
        r = to_dev(synth.complex_field((B, *ctx.grid_shape()), 21))
        want = ctx.precondition(r)
    with gpu_context(nmap, levels=3, max_batch=REP * B, restart=1) as ctx:
        got = ctx.precondition(r.repeat(REP, 1, 1))
    assert bool((got.view(REP, *want.shape) == want).all())
